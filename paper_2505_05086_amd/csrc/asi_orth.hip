// Orthogonalize (Alg. 1): Q factor of the thin QR of P with positive diagonal R, in fp64.
//
// Method: Cholesky-QR with a diagonal shift on the first pass (safe for cond(P) up to
// ~1e9, far beyond what a Gram matrix alone allows), followed by plain Cholesky-QR:
//     pass 0: G = P^T P + s I = R0^T R0,  Q0 = P R0^-1        cond(Q0) ~ 1e3
//     pass 1: G = Q0^T Q0     = R1^T R1,  Q  = Q0 R1^-1       |Q^T Q - I| ~ 1e-16 cond(Q0)^2
// cond(P) reaches (sigma_1/sigma_r)^2 * cond(U^T U_prev) ~ 1e8 on the benchmark tensors.  Q
// is handed back in fp32, so two passes are enough; the slow path below runs a third.  The
// product R1 R0 is upper triangular with a positive diagonal, so Q is the unique factor
// Gram-Schmidt produces.  Its diagonal is the norm each column keeps after the earlier ones
// are projected out; a column keeping less than 1e-12 ||P||_F is reported through *info.
//
// Fast path (r <= 64), two launches that serve all modes of a tensor at once:
//   gram0 : row slices of 16 rows sum the split partial sums of P -> P64 and write their slice Gram (fp64 MFMA); of a mode of more than
//           12 slices, groups of them are added by the workgroup of the group that arrives last.
//   apply : EVERY workgroup adds the matrices up and factors the sum: Cholesky in the registers of one wave without a shift,
//           with the shift only if a pivot is lost.  It then inverts R and bounds what one pass leaves of |Q^T Q - I|: with X = R^-1 and
//           c = max_j sum_i sqrt(G_ii) |X_ij|  (the column-scaled condition number), rounding of G, of the factor and of
//           the products gives  |Q^T Q - I| <= u ((18 + slices of a group + groups + 2 r) c^2 + 4 r c).  Below OP_DONE_TOL
//           (c up to about 2000) the first pass is certified: always where the basis has settled (c 1..300), and on
//           activations that move a little every step for most modes, but not for long modes of steep spectra (256 to 960
//           channels: c 1000 to 9000), although what one pass leaves there is 4e-9.
//           Certified: Q = P X, X still in registers.  Otherwise: Q0 = P R^-1 by block forward substitution (fp64 MFMA), written in
//           fp64 and as the fp32 result, plus the slice Gram of Q0; the last-arriving workgroup measures |Q0^T Q0 - I| and only if
//           that exceeds OP_DONE_TOL runs the second pass by itself.
// The two launches are a chain of dependent round trips to memory and of pivots.  960 x 40 (60 slices) and three short modes: 24.6 + 4.8
// us with the factorisation in the workgroup of gram0 that arrived last, 8.6 + 16.0 so; 256 x 32 21.8 + 3.9 -> 8.5 + 12.3, 32 x 8
// 14.1 + 4.0 -> 6.0 + 7.2.  Of the 14.6 us inside apply for 960 x 40: 1.7 kernel start and arguments, 1.5 the matrices, 0.8 to LDS, 6.0
// factor (ten panels of four pivots), 2.5 inverse, 1.4 product and the rest.
// Wide path (64 < r <= 192): separate Gram / Cholesky / apply launches on the packed triangle.
// Slow path (r > 192): one workgroup per mode, everything in global memory.
#include "asi_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"

#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int OP_RS = 32;              // rows per slice of apply
constexpr int OP_GS = 16;              // rows per slice of gram0
constexpr int OP_RMAX = 64;
constexpr int OP_ONE_GROUP = 12;       // slices of gram0 that apply adds up itself (16: 3 us dearer there, 2.7 cheaper in gram0)
constexpr int OP_LD = OP_RMAX + 1;
constexpr double OP_EPS = 1.1102230246251565e-16;
constexpr int OP_NT = 512, OP_NW = OP_NT / 64;
constexpr double OP_DONE_TOL = 1e-7;   // |Q0^T Q0 - I| below which the first pass is the result


__device__ __forceinline__ void flag_info(int32_t* info, int mode1, int col1) {
    if (info) atomicCAS(info, 0, mode1 * 1000 + col1);
}

// the modes of all layers of one launch
constexpr int kMaxOrthJobs = 4 * kMaxBatch;
struct OrthBatch {
    int njobs;
    int first[kMaxOrthJobs + 1];       // workgroups before job j (filled for the launches that walk slices)
    OrthJob job[kMaxOrthJobs];
};
struct PresumBatch {
    PresumJob job[kMaxOrthJobs];
    int njobs;
};
static_assert(sizeof(OrthBatch) <= 4096, "kernel argument limit");

__device__ __forceinline__ void find_job(const OrthBatch& a, int* ji, int* blk) {
    int j = 0;
    const int b = blockIdx.x;
    while (j + 1 < a.njobs && b >= a.first[j + 1]) ++j;
    *ji = j; *blk = b - a.first[j];
}

// Packed upper triangle: element (ga <= gb) of an r x r symmetric matrix
__device__ __forceinline__ int tri_idx(int r, int ga, int gb) { return ga * r - (ga * (ga - 1)) / 2 + (gb - ga); }

// What one workgroup writes for another of the same launch: stores and loads that go past the XCD's L2 (agent scope), so that
// the hand-over needs no write-back and no invalidation of whole caches.
__device__ __forceinline__ void publish(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double published(const double* p, long long idx, bool ok) {
    const double v = __hip_atomic_load(p + (ok ? idx : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return ok ? v : 0.0;
}

// Gram of the ROWS rows held in Ps (zero padded to 64 columns), added to the wave's block pairs in acc: pair `wave` and, beyond eight
// of them, pair `wave + 8` of the blocks on and above the diagonal, row by row
constexpr int OP_PAIRS = 2;
__device__ __forceinline__ void wave_pair(int nb, int pr, int* ab, int* bb) {
    int i = 0, rem = pr;
    while (i < nb && rem >= nb - i) { rem -= nb - i; ++i; }
    *ab = i; *bb = i + rem;                                  // ab == nb: no such pair
}
template <int ROWS>
__device__ __forceinline__ void gram_add(const double (*Ps)[OP_LD], int r, v4d (&acc)[OP_PAIRS]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lg = lane >> 4, ll = lane & 15;
    const int nb = (r + 15) / 16;
#pragma unroll
    for (int s = 0; s < OP_PAIRS; ++s) {
        int ab, bb;
        wave_pair(nb, wave + OP_NW * s, &ab, &bb);
        if (ab < nb)                                         // uniform
#pragma unroll
            for (int ks = 0; ks < ROWS / 4; ++ks)
                acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(Ps[4 * ks + lg][16 * ab + ll], Ps[4 * ks + lg][16 * bb + ll], acc[s], 0, 0, 0);
    }
}
// -> packed upper triangle Gout (r (r+1) / 2)
__device__ __forceinline__ void gram_publish(const v4d (&acc)[OP_PAIRS], int r, double* Gout) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lg = lane >> 4, ll = lane & 15;
    const int nb = (r + 15) / 16;
#pragma unroll
    for (int s = 0; s < OP_PAIRS; ++s) {
        int ab, bb;
        wave_pair(nb, wave + OP_NW * s, &ab, &bb);
        if (ab < nb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int ga = 16 * ab + lg + 4 * v, gb = 16 * bb + ll;
                if (ga < r && gb < r && ga <= gb) publish(Gout + tri_idx(r, ga, gb), acc[s][v]);
            }
    }
}

// ---- first level of the partial-sum tree -----------------------------------------------------
// When a mode arrives with more than 32 split partial sums, groups of 32 are added first
// (fixed order inside a group), so that no workgroup of gram0 has to walk hundreds of them.
__global__ __launch_bounds__(256) void k_orth_presum(PresumBatch a) { presum_block(a.job, a.njobs, blockIdx.x); }

// ---- chol -----------------------------------------------------------------------------------
__device__ __forceinline__ double bcast_lane(double x, int src) {      // src uniform
    const int lo = __builtin_amdgcn_readlane(__double2loint(x), src);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(x), src);
    return __hiloint2double(hi, lo);
}

// e / r for 0 <= e < 2^16 and 1 <= r <= 192 without an integer division: the rounded float quotient
// of (e + 0.5) is exact in that range (the same device as in the product kernels).
__device__ __forceinline__ int small_div(int e, float inv_r) { return (int)(((float)e + 0.5f) * inv_r); }

// The matrix is reached through an accessor (ld(row, col), st(row, col, value)): a square LDS array
// for r <= 64, the packed upper triangle for wider matrices.  Only entries with row <= col are used.
struct GramSquare {
    double (*Gs)[OP_LD];
    __device__ __forceinline__ double ld(int row, int col) const { return Gs[row][col]; }
    __device__ __forceinline__ void st(int row, int col, double v) const { Gs[row][col] = v; }
};
struct GramPacked {                      // row-wise packed upper triangle of an r x r matrix, identity beyond r
    double* Gp;
    int r;
    __device__ __forceinline__ int idx(int row, int col) const { return row * r - (row * (row - 1)) / 2 + (col - row); }
    __device__ __forceinline__ double ld(int row, int col) const {
        const bool in = row <= col && col < r;
        const double v = Gp[in ? idx(row, col) : 0];
        return in ? v : (row == col ? 1.0 : 0.0);
    }
    __device__ __forceinline__ void st(int row, int col, double v) const {
        if (row <= col && col < r) Gp[idx(row, col)] = v;
    }
};
// Cholesky on the fp64 MFMA by ONE wave, four pivots per round.  A 16 x 16 block sits in the MFMA's result layout: register v
// of lane (lg, ll) is element (4 v + lg, ll), so panel p of four rows is register p of every lane, and as it is both the A
// operand (element (k, i) of the panel, k = lg) and the B operand of a rank-4 update.  A round fetches the panel's 4x4
// diagonal block D = L4 diag(q) L4^T with v_readlane and factors it redundantly in every lane; the panel's rows become
// W = L4^-1 G_panel (one product per block), the rows below lose W^T diag(1/q) W (another).  An identity block that goes through
// the same row operations becomes the inverse of the block's unit lower triangular factor.
// Rows are left unscaled: row k holds R[k][j] * R[k][k], the diagonal the pivots R[k][k]^2.
// A non-positive pivot is replaced (by a number in [1, 2)) and reported through `bad` (1-based index, first one wins).
struct Panel4 {
    double li;           // lane (lg, ll): element [ll mod 4][lg] of L4^-1
    double pl;           // 1 / q of row lg of the panel
};
// g: the panel's register of the diagonal block; p: the panel's number in the block; col1: 1-based index of its first pivot
__device__ __forceinline__ Panel4 factor_panel(double g, int p, int col1, int lg, int ll, int* bad) {
    double a[4][4], pi[4], m[4][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
        for (int k2 = k; k2 < 4; ++k2) a[k][k2] = bcast_lane(g, 16 * k + 4 * p + k2);
    // column lg of L4^-1 by forward substitution, beside the pivots
    double x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = lg == k ? 1.0 : 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        double q = a[k][k];
        const bool okp = q > 0.0;                        // false for zero, negative, NaN
        *bad = (!okp && *bad == 0) ? col1 + k : *bad;
        q = __hiloint2double(okp ? __double2hiint(q) : 0x3ff00000, __double2loint(q));
        double inv = __builtin_amdgcn_rcp(q);
        const double e = fma(-q, inv, 1.0);              // r (1 + e + e^2): full accuracy from the estimate's 2^-20 and better
        inv = fma(inv * e, 1.0 + e, inv);
        pi[k] = inv;
#pragma unroll
        for (int k2 = k + 1; k2 < 4; ++k2) m[k][k2] = a[k][k2] * inv;                // L4[k2][k]
#pragma unroll
        for (int k2 = k + 1; k2 < 4; ++k2) {
#pragma unroll
            for (int k3 = k2; k3 < 4; ++k3) a[k2][k3] = fma(-m[k][k2], a[k][k3], a[k2][k3]);
            x[k2] = fma(-m[k][k2], x[k], x[k2]);
        }
    }
    // (pinned: left alone the compiler turns the selects into a ladder of branches around the arithmetic)
    asm volatile("" : "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(pi[0]), "+v"(pi[1]), "+v"(pi[2]), "+v"(pi[3]));
    Panel4 o;
    o.li = (ll & 2) ? ((ll & 1) ? x[3] : x[2]) : ((ll & 1) ? x[1] : x[0]);
    o.pl = (lg & 2) ? ((lg & 1) ? pi[3] : pi[2]) : ((lg & 1) ? pi[1] : pi[0]);
    return o;
}
__device__ __forceinline__ v4d mfma64(double a, double b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
// L4^-1 times four rows of 16: four 4 x 4 x 4 blocks in one instruction, operands and result in the layout of a panel (lane 16 k + 4 block
// + i holds element [i][k] of the left operand).  A dependent one takes 33 cycles where the 16 x 16 x 4 form, three quarters of
// it zeros, takes 80.
__device__ __forceinline__ double panel_rows(double li, double g) { return __builtin_amdgcn_mfma_f64_4x4x4f64(li, g, 0.0, 0, 0, 0); }

// One diagonal block of a matrix in LDS behind an accessor (wide ranks): U in place, pinvs[base+k] the pivots' reciprocals,
// Xb[i][j] = (L^-1)[j][i].
template <class GA>
__device__ void chol_block16(const GA G, double (*Xb)[17], double* pinvs, int base, int* bad_io) {
    const int lane = threadIdx.x & 63, lg = lane >> 4, ll = lane & 15;
    v4d g, x;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = 4 * v + lg;
        g[v] = G.ld(base + (i < ll ? i : ll), base + (i < ll ? ll : i));
        x[v] = i == ll ? 1.0 : 0.0;
    }
    int bad = *bad_io;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const Panel4 f = factor_panel(g[p], p, base + 4 * p + 1, lg, ll, &bad);
        const double w = panel_rows(f.li, g[p]), wx = panel_rows(f.li, x[p]);
        if (p < 3) {
            const v4d gn = mfma64(-w, w * f.pl, g), xn = mfma64(-w, wx * f.pl, x);
#pragma unroll
            for (int v = p + 1; v < 4; ++v) { g[v] = gn[v]; x[v] = xn[v]; }
        }
        g[p] = w;
        x[p] = wx;
        if (ll == 0) pinvs[base + 4 * p + lg] = f.pl;
    }
    *bad_io = bad;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int i = 4 * v + lg;
        if (i <= ll) G.st(base + i, base + ll, g[v]);
        Xb[ll][i] = x[v];
    }
}

// A matrix of nb <= NB blocks a side (r <= 64), whole, in the registers of the wave: no LDS round trip and no barrier between
// panels.  In: Gs (symmetric, identity beyond r); out: U in the upper blocks of Gs, Xs[b][i][j] = (L_bb^-1)[j][i].
// Per panel the chain is fetch, four reciprocals, two products; pivots left unchecked (the test and the replacement out of the chain)
// change nothing.
// 48 columns: 9.5 us as blocks of 16 with the block row and the trailing blocks dealt to all waves behind barriers, 7.6 so, 6.8 with the
// panel's rows multiplied in 4 x 4 blocks.  Panels wholly beyond r are rows of the identity and are skipped (40 columns: 6.0).
template <int NB>
__device__ __forceinline__ void chol_wave(double (*Gs)[OP_LD], double (*Xs)[16][17], int r, int* bad_io) {
    const int lane = threadIdx.x & 63, lg = lane >> 4, ll = lane & 15;
    const int nb = (r + 15) / 16;
    v4d g[NB][NB];
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = I; J < NB; ++J)
#pragma unroll
            for (int v = 0; v < 4; ++v) g[I][J][v] = Gs[16 * I + 4 * v + lg][16 * J + ll];
    int bad = 0;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (b < nb) {                                    // uniform
            v4d x;
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = 4 * v + lg == ll ? 1.0 : 0.0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                if (p > 0 && 16 * b + 4 * p >= r) continue;      // uniform: rows of the identity
                const Panel4 f = factor_panel(g[b][b][p], p, 16 * b + 4 * p + 1, lg, ll, &bad);
                double w[NB], mw[NB];
                w[b] = panel_rows(f.li, g[b][b][p]);
                mw[b] = w[b] * f.pl;
                if (p < 3) {
                    const v4d gn = mfma64(-w[b], mw[b], g[b][b]);
#pragma unroll
                    for (int v = p + 1; v < 4; ++v) g[b][b][v] = gn[v];
                }
                g[b][b][p] = w[b];
                const double wx = panel_rows(f.li, x[p]);
                if (p < 3) {
                    const v4d xn = mfma64(-w[b], wx * f.pl, x);
#pragma unroll
                    for (int v = p + 1; v < 4; ++v) x[v] = xn[v];
                }
                x[p] = wx;
#pragma unroll
                for (int J = b + 1; J < NB; ++J) {
                    w[J] = panel_rows(f.li, g[b][J][p]);
                    mw[J] = w[J] * f.pl;
                    if (p < 3) {
                        const v4d gn = mfma64(-w[b], mw[J], g[b][J]);
#pragma unroll
                        for (int v = p + 1; v < 4; ++v) g[b][J][v] = gn[v];
                    }
                    g[b][J][p] = w[J];
                }
#pragma unroll
                for (int I = b + 1; I < NB; ++I)
#pragma unroll
                    for (int J = I; J < NB; ++J) g[I][J] = mfma64(-w[I], mw[J], g[I][J]);
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                Xs[b][ll][4 * v + lg] = x[v];
#pragma unroll
                for (int J = b; J < NB; ++J)
                    if (J > b || 4 * v + lg <= ll) Gs[16 * b + 4 * v + lg][16 * J + ll] = g[b][J][v];
            }
        }
    }
    *bad_io = bad;
}

// One workgroup: sums the Gram matrices of a mode, adds the shift (first pass) and factors the sum, identity padded to a multiple
// of 16 (wave 0).  scal (written by the mode's workgroup that leads): [0] = trace(P^T P), [1 + k] = running product of the R
// diagonals, [65] = first bad pivot (certified: first column at the noise floor), [66] = 2 where the first pass is certified, 1
// where it was measured and found enough, else 0.
struct CholSmem {
    double Gs[OP_RMAX][OP_LD];       // the sum, then its factor (rows unscaled), then R
    double dinv[OP_RMAX];
    double rdiag[OP_RMAX];
    double pinvs[OP_RMAX];
    double gsq[OP_RMAX];
    double Xs[OP_RMAX / 16][16][17]; // inverses of L's diagonal blocks, then of R's
    double colmax[OP_NW];
    double s_trace;
    int s_bad;
};

// Sum of `count` packed matrices of T elements, in their order: element tid + OP_NT it in sum[it].  A round keeps up to 48
// loads per thread in flight (a round is one dependent trip to memory); up to eight matrices take a round of their own size, since
// what is asked for beyond the last costs as much as the matrices themselves.  PUBLISHED: by workgroups of this launch.
template <int RM>
constexpr int packed_its() { return (RM * (RM + 1) / 2 + OP_NT - 1) / OP_NT; }
template <int RM, bool PUBLISHED, int SB>
__device__ __forceinline__ void sum_packed_by(const double* src, int count, int T, double (&sum)[packed_its<RM>()]) {
    constexpr int ITS = packed_its<RM>();
    const int tid = threadIdx.x;
#pragma unroll
    for (int it = 0; it < ITS; ++it) sum[it] = 0.0;
#pragma unroll 1
    for (int b0 = 0; b0 < count; b0 += SB) {
        double t[SB][ITS];
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const double* m = src + (long long)(b0 + u < count ? b0 + u : count - 1) * T;       // uniform
#pragma unroll
            for (int it = 0; it < ITS; ++it) {
                const unsigned e = tid + OP_NT * it < T ? tid + OP_NT * it : 0;
                t[u][it] = PUBLISHED ? published(m, e, true) : m[e];
            }
        }
#pragma unroll
        for (int u = 0; u < SB; ++u)
#pragma unroll
            for (int it = 0; it < ITS; ++it) sum[it] += b0 + u < count ? t[u][it] : 0.0;
    }
}
template <int RM, bool PUBLISHED>
__device__ __forceinline__ void sum_packed(const double* src, int count, int T, double (&sum)[packed_its<RM>()]) {
    constexpr int ITS = packed_its<RM>(), SB = 48 / ITS > 24 ? 24 : 48 / ITS;
    if (SB > 8 && count <= 8) sum_packed_by<RM, PUBLISHED, 8>(src, count, T, sum);
    else sum_packed_by<RM, PUBLISHED, SB>(src, count, T, sum);
}

// Factors the sum of the nslices matrices.  First pass: PASS 0; lead: writes scal.  Second pass (one workgroup of the mode): false
// where the first was enough.  Leaves in sm: the factor in Gs, 1 / R_kk in dinv, R_kk in pinvs, the running products in rdiag, the square
// roots of the diagonal before elimination in gsq.
template <int RM, int PASS>
__device__ __forceinline__ bool chol_factor(const OrthJob& jb, bool lead, const double* slices, int nslices, int32_t* info, CholSmem& sm, bool* shifted_out) {
    double (*Gs)[OP_LD] = sm.Gs;
    double* rdiag = sm.rdiag;
    const int n = jb.n, r = jb.r, tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nb = (r + 15) / 16;
    constexpr int ITS = packed_its<RM>();
    const int T = (r * (r + 1)) / 2;
    double sum[ITS];
    // where the thread's elements lie in the matrix (worked out while the loads are on their way): row ga of the packed
    // triangle is the largest with tri_idx(r, ga, ga) <= e; the square root is off by one at most
    int grow[ITS], gcol[ITS];
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
        const int e = tid + OP_NT * it < T ? tid + OP_NT * it : 0;
        const float d = (float)(2 * r + 1);
        int ga = (int)((d - sqrtf(d * d - 8.0f * (float)e)) * 0.5f);
        ga = ga < 0 ? 0 : (ga > r - 1 ? r - 1 : ga);
        ga += (ga + 1 < r && tri_idx(r, ga + 1, ga + 1) <= e) ? 1 : 0;
        ga -= tri_idx(r, ga, ga) > e ? 1 : 0;
        grow[it] = ga; gcol[it] = ga + (e - tri_idx(r, ga, ga));
    }
    sum_packed<RM, PASS == 1>(slices, nslices, T, sum);
    // Gs = the summed Gram matrix, padded with the identity up to a multiple of 16
    auto scatter = [&]() __attribute__((always_inline)) {
        __syncthreads();
        const int pad = 16 * nb - r;                          // rows and columns r .. 16 nb - 1
        for (int e = tid; e < pad * 16 * nb; e += OP_NT) {
            const int k = r + e / (16 * nb), o = e % (16 * nb);
            Gs[k][o] = o == k ? 1.0 : 0.0;
            Gs[o][k] = o == k ? 1.0 : 0.0;
        }
#pragma unroll
        for (int it = 0; it < ITS; ++it)
            if (tid + OP_NT * it < T) {
                Gs[grow[it]][gcol[it]] = sum[it];
                Gs[gcol[it]][grow[it]] = sum[it];
            }
        __syncthreads();
    };
    scatter();
    int bad = 0;
    bool shifted = false;
    if (PASS == 1) {
        // Q0 may already be orthonormal to working accuracy (a warm-started, well-conditioned P): then
        // the second pass would only reproduce the identity, and the fp32 copy of Q0 that the solve
        // has written is the result.
        double dev = 0.0;
        const float inv_r1 = 1.0f / (float)r;
        for (int e = tid; e < r * r; e += OP_NT) {
            const int ga = small_div(e, inv_r1), gb = e - ga * r;
            dev = fmax(dev, fabs(Gs[ga][gb] - (ga == gb ? 1.0 : 0.0)));
        }
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) dev = fmax(dev, __shfl_xor(dev, m));
        if (lane == 0) rdiag[wave] = dev;
        __syncthreads();
        dev = 0.0;
#pragma unroll
        for (int w = 0; w < OP_NW; ++w) dev = fmax(dev, rdiag[w]);
        __syncthreads();
        const bool done = dev <= OP_DONE_TOL;
        if (tid == 0) jb.scal[66] = done ? 1.0 : 0.0;
        if (done) {
            if (tid < 64) {
                const double floor_ = 1e-12 * sqrt(jb.scal[0]);
                const bool low = tid < r && !(jb.scal[1 + tid] > floor_);
                const unsigned long long mask = __ballot(low);
                if (tid == 0 && info) {
                    const double badv = jb.scal[65];
                    if (badv != 0.0) flag_info(info, jb.mode1, (int)badv);
                    if (mask) flag_info(info, jb.mode1, __ffsll((long long)mask));
                }
            }
            return false;
        }
        if (tid == 0) sm.s_trace = jb.scal[0];
    } else if (wave == 1) {                                   // (beside the factorisation, which is wave 0's)
        const double g = (lane < r) ? Gs[lane][lane] : 0.0;
        double tr = g;
#pragma unroll
        for (int m = 32; m >= 1; m >>= 1) tr += __shfl_xor(tr, m);
        if (lane == 0) { sm.s_trace = tr; if (lead) jb.scal[0] = tr; }
    }
    // First pass: plain Cholesky first; if a pivot is lost (non-positive, or below 1e-12 of its
    // diagonal entry: cond(P) beyond ~1e6) the factorisation is redone with the diagonal shift
    // that makes it safe up to cond(P) ~ 1e9.  The second pass factors once.
    double gdiag = 0.0;                                       // wave 0: the diagonal before elimination (unshifted)
    if (wave == 0) gdiag = lane < r ? Gs[lane][lane] : 0.0;
    for (int attempt = 0;; ++attempt) {
        if (PASS == 0) __syncthreads();                       // (the trace's reads come before the factor's writes)
        if (wave == 0) {
            chol_wave<RM / 16>(Gs, sm.Xs, r, &bad);
            const bool lost = PASS == 0 && lane < r && !(Gs[lane][lane] > 1e-12 * gdiag);
            const unsigned long long mask = __ballot(lost);
            if (lane == 0) sm.s_bad = (bad != 0 || mask != 0) ? 1 : 0;
        }
        __syncthreads();
        if (PASS != 0 || attempt != 0 || !sm.s_bad) break;
        shifted = true;
        scatter();
        if (tid < r) Gs[tid][tid] += 11.0 * ((double)n * r + (double)r * (r + 1)) * OP_EPS * sm.s_trace;
    }
    __syncthreads();
    if (tid == 0) sm.s_bad = bad;
    if (tid < r) {
        double p = Gs[tid][tid];
        if (!(p > 0.0)) p = 1.0;
        const double d = sqrt(p);
        sm.dinv[tid] = 1.0 / d;
        sm.pinvs[tid] = d;
        const double rd = (PASS == 0 ? 1.0 : jb.scal[1 + tid]) * d;
        rdiag[tid] = rd;
        if (lead) jb.scal[1 + tid] = rd;
    } else if (tid < OP_RMAX) {
        sm.dinv[tid] = 1.0; sm.pinvs[tid] = 1.0;
    }
    if (tid < OP_RMAX) sm.gsq[tid] = tid < r ? sqrt(gdiag) : 0.0;
    __syncthreads();
    *shifted_out = shifted;
    return true;
}

// X = R^-1, a wave its block column J = wave mod 4 from the diagonal block up:  X_IJ = -X_II sum_{I < K <= J} R_IK X_KJ.  A result
// block (lane: rows lg + 4 v, column ll) is the B operand of the next product as it is, K slot (v, lg) being row lg + 4 v, so
// the chain stays in registers, and so does X for the product with P.  Returns the bound on |Q^T Q - I| after one pass.
template <int RM>
__device__ __forceinline__ double invert(int r, int per_group, int nslices, CholSmem& sm, v4d (&X)[RM / 16]) {
    const int tid = threadIdx.x, nb = (r + 15) / 16;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lg = lane >> 4, ll = lane & 15, J = wave & 3;
    double cs = 0.0;                         // this lane's share of its column's sum_i sqrt(G_ii) |X_ij|
#pragma unroll
    for (int I = 0; I < RM / 16; ++I) X[I] = (v4d){0.0, 0.0, 0.0, 0.0};
    if (J < nb) {
#pragma unroll
        for (int I = RM / 16 - 1; I >= 0; --I) {
            if (I > J) continue;             // uniform
            if (I == J) {
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = lg + 4 * v;
                    X[I][v] = (ll >= i && 16 * J + ll < r) ? sm.Xs[I][i][ll] * sm.dinv[16 * J + ll] : 0.0;
                }
            } else {
                v4d acc = {0.0, 0.0, 0.0, 0.0};
                const double di = sm.dinv[16 * I + ll];
#pragma unroll
                for (int K = I + 1; K < RM / 16; ++K)
                    if (K <= J)              // uniform
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            acc = mfma64(sm.Gs[16 * I + ll][16 * K + lg + 4 * v] * di, X[K][v], acc);
                v4d o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int k = lg + 4 * v;
                    o = mfma64(k >= ll ? -sm.Xs[I][ll][k] * sm.dinv[16 * I + k] : 0.0, acc[v], o);
                }
                X[I] = o;
            }
#pragma unroll
            for (int v = 0; v < 4; ++v) cs += sm.gsq[16 * I + lg + 4 * v] * fabs(X[I][v]);
        }
        cs += __shfl_xor(cs, 16);
        cs += __shfl_xor(cs, 32);
#pragma unroll
        for (int m = 8; m >= 1; m >>= 1) cs = fmax(cs, __shfl_xor(cs, m));
    }
    if (lane == 0) sm.colmax[wave] = cs;
    __syncthreads();
    double c = 0.0;
#pragma unroll
    for (int w = 0; w < OP_NW; ++w) {
        const double m = sm.colmax[w];
        c = m > c || m != m ? m : c;         // (a NaN stays)
    }
    // (16 products in a chain per slice, the slices of a group, the groups; then factor, inverse and product)
    return OP_EPS * ((18.0 + per_group + nslices + 2.0 * r) * c * c + 4.0 * r * c);
}

// For the solve: R in the place of its factor (rows scaled by 1 / R[k][k], zeros below the diagonal and beyond r), and the inverses
// of its diagonal blocks, (R_bb^-1)[i][j] = (L_bb^-1)[j][i] / R[j][j]
template <int RM>
__device__ __forceinline__ void finish_r(int r, CholSmem& sm) {
    const int tid = threadIdx.x, gb = tid & 63, nb = (r + 15) / 16;
    double gv[RM / OP_NW];
    constexpr int DI = (RM * 16 + OP_NT - 1) / OP_NT;
    double dv[DI];
#pragma unroll
    for (int it = 0; it < RM / OP_NW; ++it) {
        const int ga = (tid >> 6) + OP_NW * it;
        const double g = sm.Gs[ga][gb] * sm.dinv[ga];
        gv[it] = (ga < r && gb < r) ? (ga < gb ? g : (ga == gb ? sm.pinvs[ga] : 0.0)) : 0.0;
    }
#pragma unroll
    for (int u = 0; u < DI; ++u) {
        const int e = tid + OP_NT * u, b = e >> 8, i = (e >> 4) & 15, jj = e & 15, base = 16 * b;
        const bool in = b < nb && base + i < r && base + jj < r && jj >= i;
        dv[u] = in ? sm.Xs[b][i][jj] * sm.dinv[base + jj] : 0.0;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < RM / OP_NW; ++it) sm.Gs[(tid >> 6) + OP_NW * it][gb] = gv[it];
#pragma unroll
    for (int u = 0; u < DI; ++u) {
        const int e = tid + OP_NT * u;
        if (e < nb * 256) sm.Xs[e >> 8][(e >> 4) & 15][e & 15] = dv[u];
    }
    __syncthreads();
}

// ---- hand-over from the slices of a mode to its factorisation ------------------------------
// Every workgroup of a mode calls this after its global writes.  Returns true in exactly one of
// them, the one that arrives last; by then the writes of all the others are visible to it: what was published to loads of
// the same kind, and with FENCE everything to everything.  The counter must be zero before the launch and is zero again
// afterwards.
template <bool FENCE>
__device__ bool last_arrival(int32_t* ctr, int nblk, int* s_flag) {
    if (FENCE) __threadfence();            // this thread's writes are visible device-wide ...
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // (published ones once they are acknowledged)
    __syncthreads();                       // ... for every thread of the workgroup
    if (threadIdx.x == 0) {
        const int ticket = atomicAdd(ctr, 1);
        *s_flag = (ticket == nblk - 1);
        if (ticket == nblk - 1) *ctr = 0;
    }
    __syncthreads();
    const bool last = *s_flag != 0;
    if (FENCE && last) __threadfence();    // order the reads below after the other workgroups' arrivals
    return last;
}

// ---- gram0 ----------------------------------------------------------------------------------
// A slice is 16 rows, so that the partial sums of P (5 MB for 16 splits of 960 x 40) are read by as many CUs as there are
// slices, because what one CU can read past its L2 is 25 bytes a cycle; beyond 12 slices the Grams of about sqrt(slices) of them are
// added up by the workgroup of the group that arrives last, so that the next launch finds a dozen matrices at most (sixty: 390 KB
// for each of its workgroups).
// RM bounds the ranks of the launch's modes: a slice has at most 16 * RM elements, ITS per thread.  Up to 32 a CU holds two
// workgroups (128 registers).
template <int RM>
__global__ __launch_bounds__(OP_NT, RM <= 32 ? 4 : 2) void k_orth_gram0(OrthBatch a) {
    __shared__ double Ps[OP_GS][OP_LD];
    __shared__ int s_last;
    int ji, blk;
    find_job(a, &ji, &blk);
    const OrthJob& jb = a.job[ji];
    const int n = jb.n, r = jb.r, ns = jb.nsplit, tid = threadIdx.x;
    if (blk == 0 && tid == 0 && jb.info) *jb.info = 0;            // nothing has reported yet
    const int i0 = blk * OP_GS;
    const int nrows = (n - i0 < OP_GS) ? n - i0 : OP_GS;
    const long long cnt = (long long)n * r;
    const int E = nrows * r;
    // Sum of the split partial sums, in their order; up to 32 loads per thread in flight
    constexpr int ITS = (OP_GS * RM + OP_NT - 1) / OP_NT, SB = 32 / ITS;
    double sum[ITS];
#pragma unroll
    for (int it = 0; it < ITS; ++it) sum[it] = 0.0;
#pragma unroll 1
    for (int sp0 = 0; sp0 < ns; sp0 += SB) {
        double t[SB][ITS];
#pragma unroll
        for (int u = 0; u < SB; ++u) {
            const double* src = jb.part + (long long)(sp0 + u < ns ? sp0 + u : ns - 1) * cnt + (long long)i0 * r;    // uniform
#pragma unroll
            for (int it = 0; it < ITS; ++it) t[u][it] = src[(unsigned)(tid + OP_NT * it < E ? tid + OP_NT * it : 0)];
        }
#pragma unroll
        for (int u = 0; u < SB; ++u)
#pragma unroll
            for (int it = 0; it < ITS; ++it) sum[it] += sp0 + u < ns ? t[u][it] : 0.0;
    }
    for (int e = tid; e < OP_GS * OP_LD; e += OP_NT) (&Ps[0][0])[e] = 0.0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ITS; ++it) {
        const int idx = tid + OP_NT * it;
        if (idx < E) {
            jb.P64[(long long)i0 * r + idx] = sum[it];
            const int pi = small_div(idx, 1.0f / (float)r);
            Ps[pi][idx - pi * r] = sum[it];
        }
    }
    __syncthreads();
    const int T = (r * (r + 1)) / 2, nsl = (n + OP_GS - 1) / OP_GS, gsz = jb.gsz, ngrp = (nsl + gsz - 1) / gsz;
    v4d acc[OP_PAIRS];
#pragma unroll
    for (int u = 0; u < OP_PAIRS; ++u) acc[u] = (v4d){0.0, 0.0, 0.0, 0.0};
    gram_add<OP_GS>(Ps, r, acc);
    gram_publish(acc, r, jb.Gpart + (long long)blk * T);
    if (ngrp == 1) return;
    // the workgroup that finishes a group's last slice adds the group up
    const int grp = blk / gsz, in_grp = nsl - grp * gsz < gsz ? nsl - grp * gsz : gsz;
    if (!last_arrival<false>(jb.ctr + 2 + grp, in_grp, &s_last)) return;
    double gs[packed_its<RM>()];
    sum_packed<RM, true>(jb.Gpart + (long long)grp * gsz * T, in_grp, T, gs);
#pragma unroll
    for (int it = 0; it < packed_its<RM>(); ++it)
        if (tid + OP_NT * it < T) jb.Gpart[(long long)(nsl + grp) * T + tid + OP_NT * it] = gs[it];
}

// ---- apply ----------------------------------------------------------------------------------
// One 32-row slice: P64[slice] <- P64[slice] R^-1, R and the inverses of its diagonal blocks in sm; waves 0 and 1 solve 16 rows each.
// The first pass stores the result in fp64 for the second pass and its fp32 copy in Uout (the result if the first pass turns
// out to be enough) and leaves it in Ps; the final pass stores fp32 only.
template <int RM>
__device__ void apply_slice(const OrthJob& jb, int slice, int final_pass, double (*Ps)[OP_LD], const CholSmem& sm) {
    const double (*Rs)[OP_LD] = sm.Gs;
    const double (*Ds)[16][17] = sm.Xs;
    const int n = jb.n, r = jb.r, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    const int nb = (r + 15) / 16;
    const int i0 = slice * OP_RS;
    const int nrows = (n - i0 < OP_RS) ? n - i0 : OP_RS;
    constexpr int PI = OP_RS * RM / OP_NT;
    const float inv_r = 1.0f / (float)r;
    double tp[PI];
#pragma unroll
    for (int u = 0; u < PI; ++u) {
        const int idx = u * OP_NT + tid;
        tp[u] = ldg_f64(jb.P64, (long long)i0 * r + idx, idx < nrows * r);
    }
    __syncthreads();                                      // (the last slice has been read)
    for (int e = tid; e < OP_RS * OP_LD; e += OP_NT) (&Ps[0][0])[e] = 0.0;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PI; ++u) {
        const int idx = u * OP_NT + tid;
        const int pi = small_div(idx, inv_r);
        if (idx < nrows * r) Ps[pi][idx - pi * r] = tp[u];
    }
    __syncthreads();
    // wave w < 2 owns rows 16w..16w+15 of the slice; block columns are solved left to right
    const int rw = 16 * (wave & 1);
    for (int b = 0; b < nb; ++b) {
        if (wave < 2) {
            // T = P_b - sum_{a<b} Q_a R_ab
            v4d acc = {0.0, 0.0, 0.0, 0.0};
            for (int ab = 0; ab < b; ++ab)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Ps[rw + ll][16 * ab + 4 * ks + lg],
                                                               Rs[16 * ab + 4 * ks + lg][16 * b + ll], acc, 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; ++v) Ps[rw + lg + 4 * v][16 * b + ll] -= acc[v];
        }
        __syncthreads();
        v4d q = {0.0, 0.0, 0.0, 0.0};
        if (wave < 2) {
            // Q_b = T R_bb^-1
#pragma unroll
            for (int ks = 0; ks < 4; ++ks)
                q = __builtin_amdgcn_mfma_f64_16x16x4f64(Ps[rw + ll][16 * b + 4 * ks + lg], Ds[b][4 * ks + lg][ll], q, 0, 0, 0);
        }
        __syncthreads();
        if (wave < 2) {
#pragma unroll
            for (int v = 0; v < 4; ++v) Ps[rw + lg + 4 * v][16 * b + ll] = q[v];
        }
        __syncthreads();
    }
    for (int idx = tid; idx < nrows * r; idx += OP_NT) {
        const int pi = small_div(idx, inv_r);
        const double q0 = Ps[pi][idx - pi * r];
        if (!final_pass) jb.P64[(long long)i0 * r + idx] = q0;
        jb.Uout[(long long)i0 * r + idx] = (float)q0;
    }
}

// The rest of the orthonormalisation in one launch.  EVERY workgroup of a mode adds up the mode's Gram matrices, factors the sum and
// inverts the factor for itself (the same bits in all of them), then takes its runs of slices of 32 rows: a dozen microseconds of one wave's
// dependent pivots cost nothing on a chip that has nothing else to do, and no workgroup waits for another.  One workgroup that
// arrived last did it before, inside gram0: a second level of hand-over, loads past the L2, and the factor's way through memory.
// Certified: Q = P X, wave (half h, block column J) 16 rows times its block column of X, the rows requested when the kernel starts.
// Otherwise: solve, slice Gram; the workgroup that finishes a mode's last slice checks Q0^T Q0 against the identity and, only
// if that fails, factors it and solves all slices of the mode once more by itself (a rare, slow path: it trades a launch per
// call for serial work on ill-conditioned inputs).  Its Grams lie where nothing of this launch is read: over gram0's slice
// Grams where those have been added up by groups, behind them otherwise.
template <int RM>
__global__ __launch_bounds__(OP_NT) void k_orth_apply(OrthBatch a) {
    __shared__ CholSmem sm;
    __shared__ double Ps[OP_RS][OP_LD];
    __shared__ int s_last;
    int ji, blk;
    find_job(a, &ji, &blk);
    const OrthJob& jb = a.job[ji];
    const int n = jb.n, r = jb.r, nb = (r + 15) / 16, tid = threadIdx.x;
    const int T = (r * (r + 1)) / 2, nsl = (n + OP_GS - 1) / OP_GS, ngrp = (nsl + jb.gsz - 1) / jb.gsz;
    const int mine = jb.spw * jb.rpw, first = blk * mine, nall = (n + OP_RS - 1) / OP_RS, end = first + mine < nall ? first + mine : nall;
    const int lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), J = wave & 3, h = wave >> 2;
    double av[RM / 16][4];
    auto rows = [&](int slice) __attribute__((always_inline)) {
        const int row = slice * OP_RS + 16 * h + ll;
#pragma unroll
        for (int I = 0; I < RM / 16; ++I)
            if (I <= J && J < nb)            // uniform
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int k = 16 * I + lg + 4 * v;
                    av[I][v] = jb.P64[(row < n && k < r) ? (long long)row * r + k : 0];
                }
    };
    if (RM < 64) rows(first);                // (at 64 the factorisation needs the registers)
    const bool lead = blk == 0;
    bool shifted;
    chol_factor<RM, 0>(jb, lead, jb.Gpart + (ngrp > 1 ? (long long)nsl * T : 0), ngrp > 1 ? ngrp : nsl, jb.info, sm, &shifted);
    if (!shifted) {
        v4d X[RM / 16];
        const double bound = invert<RM>(r, ngrp > 1 ? jb.gsz : 1, ngrp > 1 ? ngrp : nsl, sm, X);
        if (sm.s_bad == 0 && bound <= OP_DONE_TOL) {             // (false for NaN)
            if (lead && wave == 0) {
                const unsigned long long mask = __ballot(lane < r && !(sm.rdiag[lane] > 1e-12 * sqrt(sm.s_trace)));
                if (lane == 0) {
                    const int low = mask ? __ffsll((long long)mask) : 0;
                    jb.scal[65] = (double)low;
                    jb.scal[66] = 2.0;
                    if (low) flag_info(jb.info, jb.mode1, low);
                }
            }
            if (J >= nb) return;
            for (int s = first; s < end; ++s) {
                if (s != first || RM == 64) rows(s);
                const int row = s * OP_RS + 16 * h + ll;
                v4d q = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int I = 0; I < RM / 16; ++I)
                    if (I <= J)              // uniform
#pragma unroll
                        for (int v = 0; v < 4; ++v) q = mfma64((row < n && 16 * I + lg + 4 * v < r) ? av[I][v] : 0.0, X[I][v], q);
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int i = s * OP_RS + 16 * h + lg + 4 * v, c = 16 * J + ll;
                    if (i < n && c < r) jb.Uout[(long long)i * r + c] = (float)q[v];
                }
            }
            return;
        }
    }
    if (lead && tid == 0) { jb.scal[65] = (double)sm.s_bad; jb.scal[66] = 0.0; }
    finish_r<RM>(r, sm);
    double* second = jb.Gpart + (ngrp > 1 ? 0 : (long long)nsl * T);
    for (int run = blk * jb.rpw, s = first; s < end; ++run) {     // (a Gram matrix per run, whoever makes it: a batch gives the bits of its layers alone)
        v4d acc[OP_PAIRS];
#pragma unroll
        for (int u = 0; u < OP_PAIRS; ++u) acc[u] = (v4d){0.0, 0.0, 0.0, 0.0};
        for (int left = jb.spw; left > 0 && s < end; --left, ++s) {
            apply_slice<RM>(jb, s, 0, Ps, sm);
            gram_add<OP_RS>(Ps, r, acc);
        }
        gram_publish(acc, r, second + (long long)run * T);
    }
    if (!last_arrival<true>(jb.ctr + 1, (jb.nblk + jb.rpw - 1) / jb.rpw, &s_last)) return;
    if (!chol_factor<RM, 1>(jb, true, second, jb.nblk, jb.info, sm, &shifted)) return;
    if (tid < 64) {
        // first column (if any) whose accumulated R diagonal fell to the noise floor
        const unsigned long long mask = __ballot(tid < r && !(sm.rdiag[tid] > 1e-12 * sqrt(sm.s_trace)));
        if (tid == 0) {
            double badv = jb.scal[65];
            if (badv == 0.0 && sm.s_bad) badv = (double)sm.s_bad;
            jb.scal[65] = badv;
            if (badv != 0.0) flag_info(jb.info, jb.mode1, (int)badv);
            if (mask) flag_info(jb.info, jb.mode1, __ffsll((long long)mask));
        }
    }
    finish_r<RM>(r, sm);
    for (int s = 0; s < nall; ++s) {
        __threadfence();                   // every slice of Q0 is read back from memory
        apply_slice<RM>(jb, s, 1, Ps, sm);
    }
}

// ---- wide path, 64 < r <= 192 -----------------------------------------------------------------
// Same two passes.  The Gram matrix no longer fits the statically sized LDS arrays, so
//   gramw : 64-row blocks read P64 in 32-row sub-slices and keep their block pairs in registers
//   cholw : one workgroup per mode, Gram matrix packed (upper triangle) in up to 150 KB of
//           dynamic LDS, same right-looking factorisation
//   applyw: 32-row blocks, R's off-diagonal blocks are read straight from global memory
constexpr int OW_RMAX = 192;
constexpr int OW_LD = OW_RMAX + 1;
constexpr int OW_ROWS = 64;             // rows per gramw block
constexpr int OW_PARTS = 4;             // workgroups (blockIdx.y) that share the block pairs of a slice
constexpr int OW_MAXPAIR = 5;           // block pairs per wave: ceil(78 / (4 OW_PARTS))

// 64-row slices of a 3072-row mode are 48 workgroups with 78 block pairs each: 20 us of matrix time per wave behind three rounds
// of loads.  The pairs of a slice are dealt to four workgroups instead, each of which reads the whole slice (100 KB, from
// L2) with every load of 32 rows in flight; there are no more partial matrices to add than before.  36 -> 11 us.
__global__ __launch_bounds__(256) void k_orthw_gram(OrthBatch a) {
    __shared__ double Ps[OP_RS][OW_LD];
    int ji, blk;
    find_job(a, &ji, &blk);
    const OrthJob& jb = a.job[ji];
    const int n = jb.n, r = jb.r, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    const int nb = (r + 15) / 16, npairs = nb * (nb + 1) / 2;
    const int first = blockIdx.y + OW_PARTS * wave;         // this wave's pairs: first + 4 OW_PARTS s
    const double* __restrict__ P64 = jb.P64;
    int ab[OW_MAXPAIR], bb[OW_MAXPAIR];
#pragma unroll
    for (int s = 0; s < OW_MAXPAIR; ++s) {
        const int pr = first + 4 * OW_PARTS * s;
        int i = 0, rem = pr < npairs ? pr : 0;
        while (rem >= nb - i) { rem -= nb - i; ++i; }
        ab[s] = i; bb[s] = i + rem;
    }
    v4d acc[OW_MAXPAIR];
#pragma unroll
    for (int s = 0; s < OW_MAXPAIR; ++s) acc[s] = (v4d){0.0, 0.0, 0.0, 0.0};
    const float inv_rf = 1.0f / (float)r;
    for (int e = tid; e < OP_RS * (16 * nb - r); e += 256) Ps[e & (OP_RS - 1)][r + e / OP_RS] = 0.0;
    const int row_beg = blk * OW_ROWS;
    const int row_end = (row_beg + OW_ROWS < n) ? row_beg + OW_ROWS : n;
    for (int i0 = row_beg; i0 < row_end; i0 += OP_RS) {
        const int nrows = (row_end - i0 < OP_RS) ? row_end - i0 : OP_RS;
        double t[OP_RS * OW_RMAX / 256];
#pragma unroll
        for (int u = 0; u < OP_RS * OW_RMAX / 256; ++u) {
            const int idx = u * 256 + tid;
            t[u] = P64[(long long)i0 * r + (idx < nrows * r ? idx : 0)];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < OP_RS * OW_RMAX / 256; ++u) {
            const int idx = u * 256 + tid, row = small_div(idx, inv_rf);
            if (idx < OP_RS * r) Ps[row][idx - row * r] = idx < nrows * r ? t[u] : 0.0;      // rows past nrows become zero
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < OW_MAXPAIR; ++s) {
            if (first + 4 * OW_PARTS * s < npairs) {
                double av[OP_RS / 4], bv[OP_RS / 4];
#pragma unroll
                for (int ks = 0; ks < OP_RS / 4; ++ks) {
                    av[ks] = Ps[4 * ks + lg][16 * ab[s] + ll];
                    bv[ks] = Ps[4 * ks + lg][16 * bb[s] + ll];
                }
#pragma unroll
                for (int ks = 0; ks < OP_RS / 4; ++ks) acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[ks], bv[ks], acc[s], 0, 0, 0);
            }
        }
    }
    double* Gout = jb.Gpart + (long long)blk * r * r;
#pragma unroll
    for (int s = 0; s < OW_MAXPAIR; ++s) {
        if (first + 4 * OW_PARTS * s < npairs) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int ga = 16 * ab[s] + lg + 4 * v, gb = 16 * bb[s] + ll;
                if (ga < r && gb < r && ga <= gb) Gout[ga * r + gb] = acc[s][v];
            }
        }
    }
}

// Sum of the slice Gram matrices of a mode and its distance from the identity, spread over the chip: the
// factorisation is one workgroup, and what it reads right after other workgroups wrote it costs it 3-5 us per
// dependent round of loads (five rounds for two partial sums of a 192 x 192 matrix: 28 us of the second pass went
// into a sum whose only use was the check that the first pass had been enough).
struct GsumBatch {
    GsumJob job[kMaxOrthJobs];
    int njobs;
};
__global__ __launch_bounds__(256) void k_orthw_gsum(GsumBatch a) {
    int j = 0, b = blockIdx.x;
    while (j + 1 < a.njobs && b >= a.job[j].nchunks) { b -= a.job[j].nchunks; ++j; }
    const GsumJob& jb = a.job[j];
    const int r = jb.r, cnt = r * r;
    const int e = b * 256 + threadIdx.x;
    double s = 0.0;
    for (int b0 = 0; b0 < jb.nblk; b0 += 32) {               // 32 slices' loads in flight, added in slice order
        double t[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) t[u] = jb.in[(long long)(b0 + u < jb.nblk ? b0 + u : jb.nblk - 1) * cnt + (e < cnt ? e : 0)];
#pragma unroll
        for (int u = 0; u < 32; ++u) s += (b0 + u < jb.nblk) ? t[u] : 0.0;
    }
    double dev = 0.0;
    if (e < cnt) {
        jb.out[e] = s;
        const int ga = e / r, gb = e - ga * r;
        if (ga <= gb) dev = fabs(s - (ga == gb ? 1.0 : 0.0));   // (only the upper triangles of the slices are written)
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) dev = fmax(dev, __shfl_xor(dev, m));
    if ((threadIdx.x & 63) == 0 && dev > 0.0) atomicMax(jb.devbits, (unsigned long long)__double_as_longlong(dev));
}

extern __shared__ double ow_dyn[];

// 512 threads: with 1024 a thread may hold 128 registers, and the diagonal-block factorisation (a column
// of 16 doubles per lane plus its panels) then spills to scratch memory: 13 us per block instead of 2.
constexpr int OWC_NT = 512, OWC_NW = OWC_NT / 64;
__global__ __launch_bounds__(OWC_NT) void k_orthw_chol(OrthBatch a, int pass, int last) {
    const OrthJob jb = a.job[blockIdx.x];
    const int n = jb.n, r = jb.r, tid = threadIdx.x;
    double* Gp = ow_dyn;                              // packed upper triangle, r (r + 1) / 2
    double* dinv = ow_dyn + (r * (r + 1)) / 2;
    double* rdiag = dinv + r;
    __shared__ double s_trace;
    __shared__ int s_bad;
    auto pidx = [r](int ga, int gb) __attribute__((always_inline)) { return ga * r - (ga * (ga - 1)) / 2 + (gb - ga); };
    __shared__ int s_lost;
    __shared__ double s_red[OWC_NW];
    if (tid == 0) { s_bad = 0; s_lost = 0; }
    // Gp = sum of the slice Grams; returns this thread's share of max |G - I|.  A round keeps 32 loads
    // per thread in flight: 4 elements x 8 slices, or 16 elements x 2 slices when a tree level has
    // already added the slices up (quotient e / r by a rounded float product: exact for r * r < 2^21).
    const float inv_rf = 1.0f / (float)r;
    auto sum_gram_t = [&](auto c_c, auto u_c) __attribute__((always_inline)) {
        constexpr int C = decltype(c_c)::value, U = decltype(u_c)::value;
        double dev = 0.0;
        for (int e0 = tid; e0 < r * r; e0 += C * OWC_NT) {
            double s[C];
#pragma unroll
            for (int c = 0; c < C; ++c) s[c] = 0.0;
            for (int b0 = 0; b0 < jb.nblk; b0 += U) {
                double t[C][U];
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int u = 0; u < U; ++u) {
                        const int e = e0 + OWC_NT * c;
                        t[c][u] = ldg_f64(jb.Gpart, (long long)(b0 + u) * r * r + e, e < r * r && b0 + u < jb.nblk);
                    }
#pragma unroll
                for (int c = 0; c < C; ++c)
#pragma unroll
                    for (int u = 0; u < U; ++u) s[c] += t[c][u];
            }
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int e = e0 + OWC_NT * c;
                const int ga = small_div(e, inv_rf), gb = e - ga * r;
                if (e < r * r && ga <= gb) {
                    Gp[pidx(ga, gb)] = s[c];
                    dev = fmax(dev, fabs(s[c] - (ga == gb ? 1.0 : 0.0)));
                }
            }
        }
        return dev;
    };
    auto sum_gram = [&]() __attribute__((always_inline)) {
        return jb.nblk <= 2 ? sum_gram_t(std::integral_constant<int, 16>{}, std::integral_constant<int, 2>{})
                            : sum_gram_t(std::integral_constant<int, 4>{}, std::integral_constant<int, 8>{});
    };
    // Blocked right-looking factorisation in place, the scheme of the r <= 64 path on the packed
    // triangle: wave 0 factors a 16x16 diagonal block in registers (chol_block16, which also leaves
    // the inverse of the block's unit triangular factor in Xs and the pivots' reciprocals in pinvs),
    // then all waves solve the block row and update the trailing blocks on fp64 MFMA.  Rows are
    // left unscaled (row k holds R[k][j] R[k][k], the diagonal the pivots R[k][k]^2).  A pivot that is
    // not above 1e-12 of its diagonal entry (rdiag holds the diagonal before elimination) sets s_lost.
    const int nb = (r + 15) / 16;
    double* pinvs = rdiag + r;                               // nb * 16
    double (*Xs)[17] = reinterpret_cast<double (*)[17]>(pinvs + nb * 16);
    const GramPacked G{Gp, r};
    const int lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    // Second pass with a summed Gram matrix: its distance from the identity has been measured by the launch that
    // summed it, and the matrix itself is read only if the pass has to be carried out.
    const bool measured = pass != 0 && jb.devbits != nullptr;
    double dev = 0.0;
    if (measured) {
        dev = __longlong_as_double((long long)*jb.devbits);
    } else {
        dev = sum_gram();
        __syncthreads();
    }
    if (pass == 0) {
        if (tid == 0 && jb.devbits) *jb.devbits = 0ull;     // the second Gram sum starts from zero
        if (tid < r) rdiag[tid] = Gp[pidx(tid, tid)];
        __syncthreads();
        if (wave == 0) {                 // trace: lanes sum every 64th diagonal entry, then a fixed-order butterfly
            double tr = 0.0;
            for (int k = lane; k < r; k += 64) tr += rdiag[k];
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) tr += __shfl_xor(tr, m);
            if (lane == 0) { s_trace = tr; jb.scal[0] = tr; }
        }
        __syncthreads();
    } else {
        // Second pass: if Q0 is orthonormal to 1e-7 already, its fp32 copy (written by the first solve)
        // is the result and the final solve returns at once.
        if (!measured) {
#pragma unroll
            for (int m = 32; m >= 1; m >>= 1) dev = fmax(dev, __shfl_xor(dev, m));
            if ((tid & 63) == 0) s_red[tid >> 6] = dev;
            __syncthreads();
            dev = 0.0;
            for (int w = 0; w < OWC_NW; ++w) dev = fmax(dev, s_red[w]);
        }
        const bool done = dev <= OP_DONE_TOL;
        if (tid == 0) {
            jb.scal[2 + OW_RMAX] = done ? 1.0 : 0.0;
            s_trace = jb.scal[0];
        }
        if (done && last && jb.info) {
            // first column whose accumulated diagonal fell to the noise floor: every thread looks at one column (one
            // thread walking all of them paid a round trip to memory per column: 29 us for 192 of them)
            const double floor_ = 1e-12 * sqrt(jb.scal[0]);
            const bool low = tid < r && !(jb.scal[1 + tid] > floor_);
            if (tid == 0) s_lost = 0x7fffffff;
            __syncthreads();
            if (low) atomicMin(&s_lost, tid);
            __syncthreads();
            if (tid == 0) {
                const double bad = jb.scal[1 + OW_RMAX];
                if (bad != 0.0) flag_info(jb.info, jb.mode1, (int)bad);
                if (s_lost != 0x7fffffff) flag_info(jb.info, jb.mode1, s_lost + 1);
            }
        }
        if (done) return;
        __syncthreads();
        if (tid == 0) s_lost = 0;
        if (measured) {
            sum_gram();
            __syncthreads();
        }
        if (tid < r) rdiag[tid] = Gp[pidx(tid, tid)];
        __syncthreads();
    }
    // First pass: plain Cholesky first; only if a pivot is lost is the Gram matrix summed again, shifted
    // and factored once more (the same policy as the r <= 64 path).  The factorisation is written once,
    // inside this loop: as a lambda called from three places it was not inlined, its captured pointers
    // went through scratch memory and every LDS access in it became a flat access.
    for (int attempt = 0;; ++attempt) {
        int bad = 0;
        if (wave == 0) chol_block16(G, Xs, pinvs, 0, &bad);
        __syncthreads();
        for (int P = 0; P < nb; ++P) {
            if (tid < 16 && 16 * P + tid < r) {
                const double p = G.ld(16 * P + tid, 16 * P + tid);          // the pivot actually used
                if (!(p > 1e-12 * rdiag[16 * P + tid])) s_lost = 1;
            }
            if (P + 1 < nb) {
                // block row P right of the diagonal:  U_PJ = L_PP^-1 G_PJ
                for (int J = P + 1 + wave; J < nb; J += OWC_NW) {
                    double bv[4];
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) bv[ks] = G.ld(16 * P + 4 * ks + lg, 16 * J + ll);
                    v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)      // A[i][k] = (L^-1)[i][k] = Xs[k][i]
                        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Xs[4 * ks + lg][ll], bv[ks], acc, 0, 0, 0);
#pragma unroll
                    for (int v = 0; v < 4; ++v) G.st(16 * P + lg + 4 * v, 16 * J + ll, acc[v]);
                }
                __syncthreads();
                // trailing blocks:  G_IJ -= U_PI^T diag(1/pivot) U_PJ,  P < I <= J.  Rows k of the panel lie
                // above both blocks, so their elements sit at roff[k] + column; a column past r reads the
                // diagonal entry instead and counts as zero.  The twelve reads of a block pair are issued
                // together (pinned: left alone, each is moved into a branch of its own and waited for there).
                int roff[4];
                double pv[4];
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) {
                    const int k = 16 * P + 4 * ks + lg;
                    roff[ks] = k * r - (k * (k + 1)) / 2;
                    pv[ks] = pinvs[k];
                }
                // Wave 0 takes the next diagonal block and factors it at once (nothing it reads is still being written, and the
                // inverse Xs of this panel has been used); the other waves share the remaining pairs, three at a
                // time, so that the reads of one run under the products of another.  192 wide: 113 -> 102 us.
                const int m = nb - P - 1, npairs = m * (m + 1) / 2;
                constexpr int NP = 3;
                for (int c0 = wave; c0 < npairs; c0 += NP * (OWC_NW - 1)) {
                    double av[NP][4], bv[NP][4], cv[NP][4];
                    int cidx[NP][4];
                    bool cin[NP][4], iin[NP], jin[NP];
#pragma unroll
                    for (int t = 0; t < NP; ++t) {
                        const int c = c0 + t * (OWC_NW - 1);
                        const bool have = c < npairs && (t == 0 || wave != 0);
                        int I = 0, rem = have ? c : 0;
                        while (rem >= m - I) { rem -= m - I; ++I; }
                        const int J = P + 1 + I + rem;
                        I += P + 1;
                        const int ci = 16 * I + ll, cj = 16 * J + ll;
                        iin[t] = ci < r; jin[t] = cj < r;
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) {
                            const int k = 16 * P + 4 * ks + lg;
                            av[t][ks] = Gp[roff[ks] + (iin[t] ? ci : k)];
                            bv[t][ks] = Gp[roff[ks] + (jin[t] ? cj : k)];
                        }
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int rw = 16 * I + lg + 4 * v;
                            cin[t][v] = have && rw <= cj && jin[t];
                            cidx[t][v] = cin[t][v] ? rw * r - (rw * (rw + 1)) / 2 + cj : 0;
                            cv[t][v] = Gp[cidx[t][v]];
                        }
                    }
#pragma unroll
                    for (int t = 0; t < NP; ++t)
#pragma unroll
                        for (int ks = 0; ks < 4; ++ks) asm volatile("" : "+v"(av[t][ks]), "+v"(bv[t][ks]), "+v"(cv[t][ks]));
                    v4d acc[NP];
#pragma unroll
                    for (int t = 0; t < NP; ++t)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[t][v] = cin[t][v] ? cv[t][v] : 0.0;
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                        for (int t = 0; t < NP; ++t)
                            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(iin[t] ? -av[t][ks] : 0.0, jin[t] ? bv[t][ks] * pv[ks] : 0.0,
                                                                          acc[t], 0, 0, 0);
#pragma unroll
                    for (int t = 0; t < NP; ++t)
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            if (cin[t][v]) Gp[cidx[t][v]] = acc[t][v];
                    if (wave == 0) break;
                }
                if (wave == 0) chol_block16(G, Xs, pinvs, 16 * (P + 1), &bad);
                __syncthreads();
            }
        }
        if (tid == 0) s_bad = bad;
        __syncthreads();
        if (pass != 0 || attempt != 0 || !(s_lost || s_bad)) break;
        __syncthreads();
        if (tid == 0) { s_bad = 0; s_lost = 0; }
        sum_gram();
        __syncthreads();
        const double shift = 11.0 * ((double)n * r + (double)r * (r + 1)) * OP_EPS * s_trace;
        if (tid < r) Gp[pidx(tid, tid)] += shift;
        __syncthreads();
    }
    if (tid < r) {
        double p = Gp[pidx(tid, tid)];
        if (!(p > 0.0)) p = 1.0;
        const double d = sqrt(p);
        dinv[tid] = 1.0 / d;
        const double rd = (pass == 0 ? 1.0 : jb.scal[1 + tid]) * d;
        rdiag[tid] = rd;
        jb.scal[1 + tid] = rd;
    }
    __syncthreads();
    for (int e = tid; e < r * r; e += OWC_NT) {      // R, and the rows scaled in place (each entry has one owner)
        const int ga = small_div(e, inv_rf), gb = e - ga * r;
        double v = 0.0;
        if (ga < gb) {
            v = Gp[pidx(ga, gb)] * dinv[ga];
            Gp[pidx(ga, gb)] = v;
        } else if (ga == gb) {
            v = 1.0 / dinv[ga];
        }
        jb.R[e] = v;
    }
    __syncthreads();
    if (tid < nb * 16) {
        const int b = tid >> 4, i = tid & 15, base = 16 * b;
        double x[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            double s = (j == i) ? 1.0 : 0.0;
#pragma unroll
            for (int k = 0; k < j; ++k) s = fma(-x[k], (base + j < r) ? Gp[pidx(base + k, base + j)] : 0.0, s);
            x[j] = (j >= i && base + j < r && base + i < r) ? s * dinv[base + j] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) jb.Dinv[(b * 16 + i) * 16 + j] = x[j];
    }
    __syncthreads();                                      // (the pivot flags are no longer read)
    if (tid == 0) s_lost = 0x7fffffff;
    __syncthreads();
    if (last && jb.info && tid < r && !(rdiag[tid] > 1e-12 * sqrt(s_trace))) atomicMin(&s_lost, tid);
    __syncthreads();
    if (tid == 0) {
        double bad = (pass == 0) ? 0.0 : jb.scal[1 + OW_RMAX];
        if (bad == 0.0 && s_bad) bad = (double)s_bad;
        jb.scal[1 + OW_RMAX] = bad;
        if (last && jb.info) {
            if (bad != 0.0) flag_info(jb.info, jb.mode1, (int)bad);
            if (s_lost != 0x7fffffff) flag_info(jb.info, jb.mode1, s_lost + 1);
        }
    }
}

__global__ __launch_bounds__(128) void k_orthw_apply(OrthBatch a, int final_pass) {
    __shared__ double Ps[OP_RS][OW_LD];
    int ji, blk;
    find_job(a, &ji, &blk);
    const OrthJob jb = a.job[ji];
    // the first pass was found to be orthonormal already: its fp32 copy is the result
    if (final_pass && jb.scal[2 + OW_RMAX] != 0.0) return;
    const int n = jb.n, r = jb.r, tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    const int nb = (r + 15) / 16;
    const int i0 = blk * OP_RS;
    const int nrows = (n - i0 < OP_RS) ? n - i0 : OP_RS;
    const float inv_rf = 1.0f / (float)r;
    {                                                 // the slice, every load of it in flight; zero beyond its rows and columns
        double t[OP_RS * OW_RMAX / 128];
        const double* __restrict__ src = jb.P64 + (long long)i0 * r;
#pragma unroll
        for (int u = 0; u < OP_RS * OW_RMAX / 128; ++u) {
            const int idx = u * 128 + tid;
            t[u] = src[idx < nrows * r ? idx : 0];
        }
        for (int e = tid; e < OP_RS * (16 * nb - r); e += 128) Ps[e & (OP_RS - 1)][r + e / OP_RS] = 0.0;
#pragma unroll
        for (int u = 0; u < OP_RS * OW_RMAX / 128; ++u) {
            const int idx = u * 128 + tid, row = small_div(idx, inv_rf);
            if (idx < OP_RS * r) Ps[row][idx - row * r] = idx < nrows * r ? t[u] : 0.0;
        }
    }
    __syncthreads();
    const int rw = 16 * wave;
    const double* __restrict__ R = jb.R;
    const double* __restrict__ Di = jb.Dinv;
    // A block column of R needs all block columns of Q before it, and its loads nothing: the operands of column b + 1 (up to
    // 44 + 4 per lane) travel while column b is multiplied.  Loaded four block rows at a time just before their
    // products, twelve columns were 30 dependent round trips to L2: 42 us for 3072 x 192, 29 so (with the slice in one round).
    constexpr int NB = OW_RMAX / 16;
    double rv[NB - 1][4], dv[4], rn[NB - 1][4], dn[4];
    auto r_load = [&](int b) __attribute__((always_inline)) {
        const int cb = 16 * b + ll < r ? 16 * b + ll : 0;           // a column past r: masked below
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dn[ks] = Di[(b * 16 + 4 * ks + lg) * 16 + ll];
#pragma unroll
        for (int u = 0; u < NB - 1; ++u)
            if (u < b) {
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) rn[u][ks] = R[(long long)(16 * u + 4 * ks + lg) * r + cb];
            }
    };
    r_load(0);
    for (int b = 0; b < nb; ++b) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) dv[ks] = dn[ks];
#pragma unroll
        for (int u = 0; u < NB - 1; ++u)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) rv[u][ks] = rn[u][ks];
        if (b + 1 < nb) r_load(b + 1);
        v4d acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int u = 0; u < NB - 1; ++u)
            if (u < b) {
#pragma unroll
                for (int ks = 0; ks < 4; ++ks)
                    acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Ps[rw + ll][16 * u + 4 * ks + lg], rv[u][ks], acc, 0, 0, 0);
            }
        const bool in = 16 * b + ll < r;
#pragma unroll
        for (int v = 0; v < 4; ++v) Ps[rw + lg + 4 * v][16 * b + ll] -= in ? acc[v] : 0.0;
        __syncthreads();
        v4d q = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
            q = __builtin_amdgcn_mfma_f64_16x16x4f64(Ps[rw + ll][16 * b + 4 * ks + lg], dv[ks], q, 0, 0, 0);
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) Ps[rw + lg + 4 * v][16 * b + ll] = q[v];
        __syncthreads();
    }
    for (int idx = tid; idx < nrows * r; idx += 128) {
        const int row = small_div(idx, inv_rf);
        const double q0 = Ps[row][idx - row * r];
        if (!final_pass) jb.P64[(long long)i0 * r + idx] = q0;
        jb.Uout[(long long)i0 * r + idx] = (float)q0;
    }
}

// ---- slow path: one workgroup per mode, global memory, three passes ---------------------------
constexpr int ORTH_NT = 512;
constexpr int ORTH_MAXR = 1024;

__global__ __launch_bounds__(ORTH_NT) void k_orth_big(OrthBatch a) {
    __shared__ double rdiag[ORTH_MAXR];
    __shared__ double s_inv;
    __shared__ double s_trace2;
    const OrthJob jb = a.job[blockIdx.x];
    const int n = jb.n, r = jb.r, tid = threadIdx.x;
    double* __restrict__ P = jb.P64;
    double* __restrict__ G = jb.Gpart;
    int32_t* info = jb.info;
    const long long cnt = (long long)n * r;
    for (long long e = tid; e < cnt; e += ORTH_NT) {
        double s = 0.0;
        for (int sp0 = 0; sp0 < jb.nsplit; sp0 += 8) {
            double t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) t[u] = ldg_f64(jb.part, (long long)(sp0 + u) * cnt + e, sp0 + u < jb.nsplit);
#pragma unroll
            for (int u = 0; u < 8; ++u) s += t[u];
        }
        P[e] = s;
    }
    for (int k = tid; k < r; k += ORTH_NT) rdiag[k] = 1.0;
    __syncthreads();
    for (int pass = 0; pass < 3; ++pass) {
        for (int e = tid; e < r * r; e += ORTH_NT) {
            const int ca = e / r, cb = e - ca * r;
            if (ca <= cb) {
                double s = 0.0;
                for (int i = 0; i < n; ++i) s = fma(P[(long long)i * r + ca], P[(long long)i * r + cb], s);
                G[ca * r + cb] = s;
            }
        }
        __syncthreads();
        if (pass == 0) {
            if (tid == 0) {
                double tr = 0.0;
                for (int k = 0; k < r; ++k) tr += G[k * r + k];
                s_trace2 = tr;
            }
            __syncthreads();
            const double shift = 11.0 * ((double)n * r + (double)r * (r + 1)) * OP_EPS * s_trace2;
            for (int k = tid; k < r; k += ORTH_NT) G[k * r + k] += shift;
            __syncthreads();
        }
        for (int k = 0; k < r; ++k) {
            if (tid == 0) {
                double p = G[k * r + k];
                if (!(p > 0.0)) {
                    flag_info(info, jb.mode1, k + 1);
                    p = 1.0;
                }
                const double d = sqrt(p);
                G[k * r + k] = d;
                rdiag[k] *= d;
                s_inv = 1.0 / d;
            }
            __syncthreads();
            for (int j = k + 1 + tid; j < r; j += ORTH_NT) G[k * r + j] *= s_inv;
            __syncthreads();
            const int m = r - k - 1;
            for (int e = tid; e < m * m; e += ORTH_NT) {
                const int ca = k + 1 + e / m, cb = k + 1 + e % m;
                if (ca <= cb) G[ca * r + cb] -= G[k * r + ca] * G[k * r + cb];
            }
            __syncthreads();
        }
        for (int i = tid; i < n; i += ORTH_NT) {
            double* row = P + (long long)i * r;
            for (int j = 0; j < r; ++j) {
                double s = row[j];
                for (int k = 0; k < j; ++k) s -= row[k] * G[k * r + j];
                row[j] = s / G[j * r + j];
            }
        }
        __syncthreads();
    }
    if (tid == 0 && info) {
        const double floor_ = 1e-12 * sqrt(s_trace2);
        for (int k = 0; k < r; ++k)
            if (!(rdiag[k] > floor_)) { flag_info(info, jb.mode1, k + 1); break; }
    }
    for (long long e = tid; e < cnt; e += ORTH_NT) jb.Uout[e] = (float)P[e];
}

// ---- host side -------------------------------------------------------------------------------
bool orth_fast_supported(int r) { return r <= OP_RMAX; }
int orth_slices(int n) { return (n + OP_RS - 1) / OP_RS; }
int orth_gram_slices(int n) { return (n + OP_GS - 1) / OP_GS; }
// slices per group: about the square root, no more than kOrthGroups groups
int orth_group_size(int n) {
    const int s = orth_gram_slices(n);
    if (s <= OP_ONE_GROUP) return s;                     // one group: apply adds the slices up itself
    if (s > kOrthGroups * kOrthGroups) return (s + kOrthGroups - 1) / kOrthGroups;
    int g = 1;
    while (g * g < s) ++g;
    return g;
}
// Slices of 32 rows in a run of apply: one, more where that makes more than 128 runs.  A mode of one group keeps
// the Grams of a second pass, one per run, behind those of the slices: four at most, so that no layer needs more scratch
// than with the first pass's factor in memory.
int orth_apply_slices(int n) {
    const int s = orth_slices(n), most = orth_groups(n) == 1 ? 4 : 128;
    return (s + most - 1) / most;
}
bool orth_wide_supported(int r) { return r > OP_RMAX && r <= OW_RMAX; }
int orth_wide_gram_blocks(int n) { return (n + OW_ROWS - 1) / OW_ROWS; }

static bool put_orth(int kind, int aux, const char* label, const OrthArgs& a, int nblocks, Item* out) {
    if (nblocks <= 0) return false;
    *out = Item();
    out->kind = kind; out->aux = aux; out->nblocks = nblocks;
    std::snprintf(out->label, sizeof(out->label), "%s", label);
    static_assert(sizeof(OrthArgs) <= kItemArgMax && sizeof(PresumArgs) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &a, sizeof(a));
    return true;
}
static int total_blocks(const OrthArgs& a) {
    int t = 0;
    for (int j = 0; j < a.njobs; ++j) t += a.job[j].nblk;
    return t;
}
static bool fast_args_ok(const OrthArgs& a) {
    if (a.njobs <= 0 || a.njobs > 4) return false;
    for (int j = 0; j < a.njobs; ++j) {
        const OrthJob& jb = a.job[j];
        if (jb.n <= 0 || jb.r <= 0 || jb.r > OP_RMAX || jb.nblk != orth_apply_wgs(jb.n) || jb.spw != orth_apply_slices(jb.n)) return false;
        if (jb.gsz != orth_group_size(jb.n) || orth_groups(jb.n) > kOrthGroups) return false;
        if (!jb.Gpart || !jb.scal || !jb.P64 || !jb.Uout || !jb.part || !jb.ctr) return false;
    }
    return true;
}
// summed: the factorisation may be handed slice Grams that a tree level has already added up (fewer of them)
static bool wide_args_ok(const OrthArgs& a, bool summed = false) {
    if (a.njobs <= 0 || a.njobs > 4) return false;
    for (int j = 0; j < a.njobs; ++j) {
        const OrthJob& jb = a.job[j];
        if (jb.n <= 0 || !orth_wide_supported(jb.r)) return false;
        if (summed ? (jb.nblk < 1 || jb.nblk > orth_wide_gram_blocks(jb.n)) : jb.nblk != orth_wide_gram_blocks(jb.n)) return false;
        if (!jb.Gpart || !jb.R || !jb.Dinv || !jb.scal || !jb.P64 || !jb.Uout) return false;
    }
    return true;
}

bool make_orth_presum(const PresumArgs& a, Item* out) {
    const int blocks = presum_blocks(a);
    if (blocks <= 0) return false;
    *out = Item();
    out->kind = IT_PRESUM; out->nblocks = blocks;
    std::snprintf(out->label, sizeof(out->label), "k_orth_presum");
    std::memcpy(out->arg, &a, sizeof(a));
    return true;
}
bool make_orthw_gsum(const GsumArgs& a, Item* out) {
    if (a.njobs <= 0 || a.njobs > 4) return false;
    long long blocks = 0;
    for (int j = 0; j < a.njobs; ++j) {
        const GsumJob& jb = a.job[j];
        if (!jb.in || !jb.out || !jb.devbits || jb.nblk < 1 || !orth_wide_supported(jb.r)) return false;
        if (jb.nchunks != (jb.r * jb.r + 255) / 256) return false;
        blocks += jb.nchunks;
    }
    *out = Item();
    out->kind = IT_ORTHW_GSUM; out->nblocks = (int)blocks;
    std::snprintf(out->label, sizeof(out->label), "k_orthw_gsum");
    static_assert(sizeof(GsumArgs) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &a, sizeof(a));
    return true;
}
bool make_orth_gram0(const OrthArgs& a, Item* out) {
    if (!fast_args_ok(a)) return false;
    int blocks = 0;
    for (int j = 0; j < a.njobs; ++j) blocks += orth_gram_slices(a.job[j].n);
    return put_orth(IT_GRAM0, 0, "k_orth_gram0", a, blocks, out);
}
bool make_orth_apply(const OrthArgs& a, Item* out) {
    return fast_args_ok(a) && put_orth(IT_APPLY, 0, "k_orth_apply", a, total_blocks(a), out);
}
bool make_orthw_gram(const OrthArgs& a, Item* out) {
    return wide_args_ok(a) && put_orth(IT_ORTHW_GRAM, 0, "k_orthw_gram", a, total_blocks(a), out);
}
bool make_orthw_chol(const OrthArgs& a, int pass, int last, Item* out) {
    return wide_args_ok(a, true) && put_orth(IT_ORTHW_CHOL, (pass ? 1 : 0) | (last ? 2 : 0), "k_orthw_chol", a, a.njobs, out);
}
bool make_orthw_apply(const OrthArgs& a, int final_pass, Item* out) {
    if (!wide_args_ok(a)) return false;
    OrthArgs b = a;                                // apply walks 32-row slices
    for (int j = 0; j < b.njobs; ++j) b.job[j].nblk = orth_slices(b.job[j].n);
    return put_orth(IT_ORTHW_APPLY, final_pass ? 1 : 0, "k_orthw_apply", b, total_blocks(b), out);
}
bool make_orth_big(const OrthArgs& a, Item* out) {
    if (a.njobs <= 0 || a.njobs > 4) return false;
    for (int j = 0; j < a.njobs; ++j)
        if (a.job[j].r > ORTH_MAXR || !a.job[j].Gpart || !a.job[j].P64 || !a.job[j].part || !a.job[j].Uout) return false;
    return put_orth(IT_ORTH_BIG, 0, "k_orth_big", a, a.njobs, out);
}

struct InitBatch {
    int32_t* p[kMaxBatch];
    int n;
};
__global__ void k_init_ctrl(InitBatch b) {
    if (threadIdx.x < b.n && b.p[threadIdx.x]) *b.p[threadIdx.x] = 0;
}
bool make_init_ctrl(int32_t* info, Item* out) {
    if (!info) return false;
    *out = Item();
    out->kind = IT_INIT; out->nblocks = 1;
    std::snprintf(out->label, sizeof(out->label), "k_init_ctrl");
    std::memcpy(out->arg, &info, sizeof(info));
    return true;
}

hipError_t launch_orth_items(const Item* const* items, int n, hipStream_t st, char* label_out) {
    if (n <= 0 || n > kMaxBatch) return hipErrorInvalidValue;
    const int kind = items[0]->kind, aux = items[0]->aux;
    if (kind == IT_INIT) {
        InitBatch b;
        b.n = n;
        for (int j = 0; j < kMaxBatch; ++j) b.p[j] = nullptr;
        for (int j = 0; j < n; ++j) std::memcpy(&b.p[j], items[j]->arg, sizeof(int32_t*));
        hipLaunchKernelGGL(k_init_ctrl, 1, 64, 0, st, b);
        return hipGetLastError();
    }
    long long blocks = 0;
    for (int j = 0; j < n; ++j) blocks += items[j]->nblocks;
    if (blocks <= 0 || blocks > 0x7fffffffLL) return hipErrorInvalidValue;
    dim3 grid((unsigned)blocks);
    if (kind == IT_PRESUM) {
        PresumBatch b;
        b.njobs = 0;
        for (int j = 0; j < n; ++j) {
            PresumArgs a;
            std::memcpy(&a, items[j]->arg, sizeof(a));
            for (int k = 0; k < a.njobs; ++k) b.job[b.njobs++] = a.job[k];
        }
        hipLaunchKernelGGL(k_orth_presum, grid, 256, 0, st, b);
        return hipGetLastError();
    }
    if (kind == IT_ORTHW_GSUM) {
        GsumBatch b;
        b.njobs = 0;
        for (int j = 0; j < n; ++j) {
            GsumArgs a;
            std::memcpy(&a, items[j]->arg, sizeof(a));
            for (int k = 0; k < a.njobs; ++k) b.job[b.njobs++] = a.job[k];
        }
        hipLaunchKernelGGL(k_orthw_gsum, grid, 256, 0, st, b);
        return hipGetLastError();
    }
    OrthBatch b;
    b.njobs = 0;
    int rmax = 0;
    for (int j = 0; j < n; ++j) {
        OrthArgs a;
        std::memcpy(&a, items[j]->arg, sizeof(a));
        for (int k = 0; k < a.njobs; ++k) {
            b.job[b.njobs++] = a.job[k];
            rmax = a.job[k].r > rmax ? a.job[k].r : rmax;
        }
    }
    b.first[0] = 0;
    for (int j = 0; j < b.njobs; ++j) b.first[j + 1] = b.first[j] + (kind == IT_GRAM0 ? orth_gram_slices(b.job[j].n) : b.job[j].nblk);
    if (kind == IT_APPLY) {
        // A workgroup takes a run; more where not all would be resident at once (two a CU up to rank 16, else one, for their registers): a second
        // filling of the chip factors everything once more.  Compress of four | eight layers of 8 x 512 x 2048 at rank 20 (324, 648 runs), apply
        // 25.3 -> 16.1 | 37.6 -> 18.3 us, all 263.0 -> 251.6 | 484.5 -> 464.0.
        const int resident = rmax <= 16 ? 512 : 256;
        int most = 1, rpw = 0, wgs;
        for (int j = 0; j < b.njobs; ++j) most = b.job[j].nblk > most ? b.job[j].nblk : most;
        do {
            ++rpw;
            wgs = 0;
            for (int j = 0; j < b.njobs; ++j) wgs += (b.job[j].nblk + rpw - 1) / rpw;
        } while (wgs > resident && rpw < most);
        for (int j = 0; j < b.njobs; ++j) {
            b.job[j].rpw = rpw;
            b.first[j + 1] = b.first[j] + (b.job[j].nblk + rpw - 1) / rpw;
        }
        grid = dim3((unsigned)wgs);
    }
    const int rm = rmax <= 16 ? 16 : (rmax <= 32 ? 32 : (rmax <= 48 ? 48 : 64));   // register shape of the fast kernels
    if (label_out && (kind == IT_GRAM0 || kind == IT_APPLY))
        std::snprintf(label_out, 96, "%s<%d>", kind == IT_GRAM0 ? "k_orth_gram0" : "k_orth_apply", rm);
    switch (kind) {
        case IT_GRAM0:
            if (rm == 16) hipLaunchKernelGGL(k_orth_gram0<16>, grid, OP_NT, 0, st, b);
            else if (rm == 32) hipLaunchKernelGGL(k_orth_gram0<32>, grid, OP_NT, 0, st, b);
            else if (rm == 48) hipLaunchKernelGGL(k_orth_gram0<48>, grid, OP_NT, 0, st, b);
            else hipLaunchKernelGGL(k_orth_gram0<64>, grid, OP_NT, 0, st, b);
            break;
        case IT_APPLY:
            if (rm == 16) hipLaunchKernelGGL(k_orth_apply<16>, grid, OP_NT, 0, st, b);
            else if (rm == 32) hipLaunchKernelGGL(k_orth_apply<32>, grid, OP_NT, 0, st, b);
            else if (rm == 48) hipLaunchKernelGGL(k_orth_apply<48>, grid, OP_NT, 0, st, b);
            else hipLaunchKernelGGL(k_orth_apply<64>, grid, OP_NT, 0, st, b);
            break;
        case IT_ORTHW_GRAM:
            hipLaunchKernelGGL(k_orthw_gram, dim3(grid.x, OW_PARTS), 256, 0, st, b);
            break;
        case IT_ORTHW_CHOL: {
            // packed triangle, dinv, rdiag, pivot reciprocals, inverse block factor
            const auto bytes = [](size_t r) { return sizeof(double) * (r * (r + 1) / 2 + 2 * r + (r + 15) / 16 * 16 + 16 * 17); };
            const size_t lds = bytes((size_t)rmax);
            static LdsAllowed allowed;
            const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_orthw_chol), bytes(OW_RMAX), allowed);
            if (e != hipSuccess) return e;
            hipLaunchKernelGGL(k_orthw_chol, grid, OWC_NT, lds, st, b, aux & 1, (aux >> 1) & 1);
            break;
        }
        case IT_ORTHW_APPLY:
            hipLaunchKernelGGL(k_orthw_apply, grid, 128, 0, st, b, aux);
            break;
        case IT_ORTH_BIG:
            hipLaunchKernelGGL(k_orth_big, grid, ORTH_NT, 0, st, b);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace asi
