// Rank-selection front end (Sec. 3.3): what has to be measured on a stored activation before training
// starts, so that ranks can be chosen per layer under a memory budget.
//
//   mode spectrum      eigenvalues (and eigenvectors) of G = A_m A_m^T, the squared singular values and
//                      left singular vectors of the mode-m unfolding (App. A.2): k_mode_gram accumulates
//                      G in fp64 on the MFMA, split over column ranges; k_gram_reduce adds the ranges in a
//                      fixed order; k_chol_panel factors it (G = R^T R), a cyclic one-sided Jacobi iteration
//                      (k_jacobi_small, k_jacobi_block, k_jacobi_one) orthogonalises the rows of W = R, after which row k
//                      is sqrt(lambda_k) v_k^T; k_spectrum_finish sorts.
//   explained variance ranks per threshold (Sec. 3.3, Step 1): k_ev_ranks.
//   perplexity         Frobenius norm of the difference of two weight gradients (Eq. 7): k_frob_partial,
//                      k_frob_final.
//   budgeted choice    Eq. 8-9 by recursive backtracking with bounds, on the host (asi_rank_select).
//
// The compressed gradient itself comes from the library's hot path (asi_core_project and
// asi_weight_grad_* on the truncated eigenvectors).
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <limits>
#include <vector>

#include "../../include/asi.h"
#include "asi_device.h"
#include "asi_lds.h"

namespace {

using namespace asi;

typedef float v4f __attribute__((ext_vector_type(4)));
typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int RK_NMAX = 512;            // longest mode the Jacobi kernel takes (8 elements per lane)
constexpr int RK_T = 64;                // Gram tile: 64 x 64 outputs, 64 unfolding columns per chunk
constexpr int RK_LD = RK_T + 4;         // LDS row pitch in floats (16 bytes more than a multiple of 128)
constexpr int RK_MAX_SPLIT = 256;
constexpr size_t RK_ALIGN = 256;
constexpr int RK_FROB_WG = 1024;

inline size_t align_up(size_t x) { return (x + RK_ALIGN - 1) / RK_ALIGN * RK_ALIGN; }

struct CholScale {
    double scale, shift;                                 // what the factorisation applied: W^T W = scale (G + shift / scale I)
    double bad;                                          // 0; G not finite: what every eigenvalue is returned as, NaN or Inf
};
// One mode of a call.  The modes of a tensor are independent and each is a long chain of small launches, so the launches serve
// all of them: workgroup b belongs to the mode j with first[j] <= b < first[j + 1].  The rank-selection row of a (128, 160, 7, 7)
// layer, one mode after the other 3620 us, so 2380 (2150 with one copy for all counters): the 128-long mode (84 launches of 11 us)
// runs beside the 160-long one (108 of 14).
struct SpecJob {
    const void* X;
    long long outer, inner, ncols;
    int n, tiles, nsplit, nchunks;
    double* part;                       // (nsplit, n, n)
    double* G;
    double* W;
    double* norms;
    CholScale* sc;
    int32_t* rot;                       // rotations of every sweep that count against convergence
    double shift_factor, tol2;
    double* lam;
    float* vec;
};
constexpr int RK_MODES = 4;
struct SpecBatch {
    int njobs;
    int first[RK_MODES + 1];
    SpecJob job[RK_MODES];
};
__device__ __forceinline__ const SpecJob& find_mode(const SpecBatch& a, int* blk) {
    const int b = blockIdx.x;
    int j = 0;
#pragma unroll
    for (int k = 1; k < RK_MODES; ++k) j += b >= a.first[k] ? 1 : 0;     // (behind the last mode: the grid's end)
    *blk = b - a.first[j];
    return a.job[j];
}

// 1 / x for normal x: the hardware's estimate (2^-20 or better) and one step of third order, which leaves one rounding (67 million random
// x from 2^-40 to 2^23: the bits of the division, in a third of its instructions)
__device__ __forceinline__ double recip64(double x) {
    const double r = __builtin_amdgcn_rcp(x), e = fma(-x, r, 1.0);
    return fma(r * e, 1.0 + e, r);
}

// One 64 x 64 tile of G over the column chunks z, z + nsplit, ...  Wave w owns rows 16 w .. 16 w + 15 of the
// tile.  Both operands come from LDS tiles held row-major (mode index x columns); a 16-byte read gives a lane
// the columns 4 lg .. 4 lg + 3 of a 16-column block, which stand for K slot lg of four MFMA steps (the same
// assignment for both operands, and a sum over columns does not care about their order).
template <typename T>
__global__ __launch_bounds__(256) void k_mode_gram(SpecBatch a) {
    int blk;
    const SpecJob& jb = find_mode(a, &blk);
    __shared__ __align__(16) float Xi[RK_T * RK_LD];
    __shared__ __align__(16) float Xj[RK_T * RK_LD];
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    const int tile = blk % (jb.tiles * jb.tiles), z = blk / (jb.tiles * jb.tiles);
    const int bi = tile / jb.tiles, bj = tile - bi * jb.tiles;
    const int n = jb.n;
    const long long inner = jb.inner, ncols = jb.ncols;
    const bool diag = bi == bj;
    const bool last = inner == 1;       // the mode index is the contiguous one: lanes run along it
    v4d acc[4];
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[b] = (v4d){0.0, 0.0, 0.0, 0.0};

    for (int ch = z; ch < jb.nchunks; ch += jb.nsplit) {
        const long long c0 = (long long)ch * RK_T;
        // tile element (row, col): 16 passes of 4 rows x 64 columns; along the last mode 64 rows x 4 columns
        float vi[16], vj[16];
        long long base0 = 0;
        bool cin0 = false;
        if (!last) {                    // this lane's column is the same in every pass
            const long long c = c0 + lane;
            cin0 = c < ncols;
            const long long cc = cin0 ? c : 0;
            const long long o = cc / inner, j = cc - o * inner;
            base0 = o * n * inner + j;
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int row = last ? lane : 4 * u + wave;
            const long long c = c0 + 4 * u + wave;               // (last mode) this pass's column; its fibre starts at c n
            const bool cin = last ? c < ncols : cin0;
            const long long base = last ? (cin ? c : 0) * n : base0;
            const int ri = bi * RK_T + row, rj = bj * RK_T + row;
            const float xi = to_f32(X[base + (long long)(ri < n ? ri : 0) * inner]);
            vi[u] = (cin && ri < n) ? xi : 0.f;
            if (!diag) {
                const float xj = to_f32(X[base + (long long)(rj < n ? rj : 0) * inner]);
                vj[u] = (cin && rj < n) ? xj : 0.f;
            } else {
                vj[u] = 0.f;
            }
        }
        __syncthreads();                // the previous chunk is no longer read
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int row = last ? lane : 4 * u + wave, col = last ? 4 * u + wave : lane;
            Xi[row * RK_LD + col] = vi[u];
            if (!diag) Xj[row * RK_LD + col] = vj[u];
        }
        __syncthreads();
        const float* bsrc = diag ? Xi : Xj;
#pragma unroll
        for (int kk = 0; kk < RK_T / 16; ++kk) {
            const v4f a4 = *reinterpret_cast<const v4f*>(Xi + (16 * wave + ll) * RK_LD + 16 * kk + 4 * lg);
            v4f b4[4];
#pragma unroll
            for (int b = 0; b < 4; ++b) b4[b] = *reinterpret_cast<const v4f*>(bsrc + (16 * b + ll) * RK_LD + 16 * kk + 4 * lg);
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const double a = (double)a4[s];
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    acc[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (double)b4[b][s], acc[b], 0, 0, 0);
            }
        }
    }
    // fp64 MFMA result layout: lane holds row lg + 4 v, column ll of its 16 x 16 block
    double* out = jb.part + (long long)z * n * n;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = bi * RK_T + 16 * wave + lg + 4 * v, j = bj * RK_T + 16 * b + ll;
            if (i < n && j < n) out[(long long)i * n + j] = acc[b][v];
        }
}

// G[e] = sum over the column ranges, in their order, 32 of them in flight; the first workgroup clears the iteration's counters
__global__ __launch_bounds__(256) void k_gram_reduce(SpecBatch a, int nzero) {
    int blk;
    const SpecJob& jb = find_mode(a, &blk);
    if (blk == 0 && (int)threadIdx.x < nzero) jb.rot[threadIdx.x] = 0;
    const double* __restrict__ part = jb.part;
    const int nsplit = jb.nsplit;
    const long long cnt = (long long)jb.n * jb.n, e = (long long)blk * 256 + threadIdx.x;
    if (e >= cnt) return;
    double s = 0.0;
    for (int z0 = 0; z0 < nsplit; z0 += 32) {
        double t[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) t[u] = part[(long long)(z0 + u < nsplit ? z0 + u : nsplit - 1) * cnt + e];
#pragma unroll
        for (int u = 0; u < 32; ++u) s += z0 + u < nsplit ? t[u] : 0.0;
    }
    jb.G[e] = s;
}

__device__ __forceinline__ double wave_sum(double x) {
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, 64);
    return x;
}

// ---- Cholesky factor of the Gram matrix --------------------------------------------------------------------
// G + s I = R^T R (R upper triangular); the iteration below runs on the rows of R, whose singular values are the square
// roots of G's eigenvalues, and not on G itself: half the spread, and a factor is already half way to orthogonal rows
// (18 sweeps become 12 on a 160-long mode whose spectrum falls over six decades and ends in noise; simulated for
// several spectra before it was built).  The shift s = (4 n + adds) u trace(G), u = 2^-53, keeps every pivot positive whatever
// G's rank: adds is the longest chain of additions behind an entry of G (the products themselves are exact), so the rounding
// of G is at most adds u sqrt(G_ii G_jj) an entry and adds u trace(G) in norm, and 4 n u trace(G) covers the
// factorisation's own.  (With 4 n u trace(G) alone, pivots of constant samples went negative: an eigenvalue of 8 samples of
// 1 M equal values each was off by 4.5e-12 of the trace, of 32 of 4 M by 2.3e-10; 5e-14 and 1.4e-13 so.)
// It is subtracted from the eigenvalues again, so it costs no accuracy beyond the rounding of G itself.  G is also
// scaled by a power of two (exact) so that its trace is near 1: the iteration squares squares.
// One launch per panel of 32 rows: workgroup (I, J) factors the 32 x 32 diagonal block (redundantly: 32 dependent steps,
// 3 us, less than a launch of its own), solves the panel's blocks above I and J and updates the trailing block (I, J).
constexpr int RK_CB = 32;

__global__ __launch_bounds__(256) void k_chol_scale(SpecBatch a) {
    int blk;
    const SpecJob& jb = find_mode(a, &blk);
    const double* __restrict__ G = jb.G;
    const int n = jb.n;
    CholScale* out = jb.sc;
    __shared__ double red[4];
    __shared__ int s_nan;
    const int tid = threadIdx.x;
    if (tid == 0) s_nan = 0;
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < RK_NMAX / 256; ++u) {
        const int k = tid + 256 * u;
        const double g = G[(long long)(k < n ? k : 0) * (n + 1)];
        s += k < n ? g : 0.0;
    }
    s = wave_sum(s);
    if ((tid & 63) == 0) red[tid >> 6] = s;
    __syncthreads();
    const double tr = (red[0] + red[1]) + (red[2] + red[3]);
    const bool finite = tr < INFINITY;                   // (the trace of squares: finite if every entry of G is)
    if (!finite) {                                       // the same for all threads
        for (int e = tid; e < n * n; e += 256)
            if (isnan(G[e])) s_nan = 1;
        __syncthreads();
    }
    if (tid == 0) {
        int e = 0;
        const bool ok = tr > 0.0 && tr < 1e300;          // (a zero tensor: the factor is sqrt(shift) I)
        if (ok) (void)frexp(tr, &e);
        out->scale = ldexp(1.0, -e);
        out->shift = ok ? jb.shift_factor * ldexp(tr, -e) : 1.0;
        out->bad = finite ? 0.0 : (s_nan ? NAN : INFINITY);
    }
}

__global__ __launch_bounds__(256) void k_chol_panel(SpecBatch a, int P) {
    int blk;
    const SpecJob& jb = find_mode(a, &blk);
    double* __restrict__ G = jb.G;
    double* __restrict__ W = jb.W;
    const CholScale* __restrict__ sc = jb.sc;
    const int n = jb.n;
    constexpr int B = RK_CB, LD = B + 1;
    __shared__ double D[B * LD], Xi[B * LD], Xj[B * LD], dinv[B];
    const int tid = threadIdx.x, nb = (n + B - 1) / B, rest = nb - P - 1;
    // workgroup 0 writes the diagonal block of R; the others are the tiles I <= J of the trailing matrix
    int I = P, J = P;
    if (rest > 0) {
        int q = blk, i = 0;
        while (q >= rest - i) { q -= rest - i; ++i; }
        I = P + 1 + i; J = I + q;
    }
    const double scale = P == 0 ? sc->scale : 1.0, shift = P == 0 ? sc->shift : 0.0;   // applied when G is first read
    auto ld = [&](int row, int col) {                    // G is symmetric; only blocks on or above the diagonal stay valid
        const bool in = row < n && col < n;
        const double g = G[(long long)(in ? row : 0) * n + (in ? col : 0)];
        return in ? g * scale + (row == col ? shift : 0.0) : (row == col ? 1.0 : 0.0);
    };
    double td[4], ti[4], tj[4], tg[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + 256 * u, r = e >> 5, c = e & 31;
        td[u] = ld(P * B + r, P * B + c);
        ti[u] = ld(P * B + r, I * B + c);
        tj[u] = ld(P * B + r, J * B + c);
        tg[u] = ld(I * B + r, J * B + c);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int e = tid + 256 * u, r = e >> 5, c = e & 31;
        D[r * LD + c] = td[u]; Xi[r * LD + c] = ti[u]; Xj[r * LD + c] = tj[u];
    }
    __syncthreads();
    // D = R_PP^T R_PP, rows left unscaled (row k holds R_kk R_kj) and the pivots' reciprocals kept: one barrier per step
    const int r0 = tid >> 5, c0 = tid & 31;
    for (int k = 0; k < B; ++k) {
        const double pk = recip64(D[k * LD + k]), dk = D[k * LD + c0] * pk;
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = D[(r0 + 8 * u) * LD + c0] - D[k * LD + r0 + 8 * u] * dk;
        if (tid == 0) dinv[k] = pk;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (r0 + 8 * u > k && c0 >= r0 + 8 * u) D[(r0 + 8 * u) * LD + c0] = v[u];
        __syncthreads();
    }
    if (rest > 0 && tid < 2 * B) {
        // forward substitution down one column of the panel (unscaled rows: x_k = g_k, later rows lose R_kr R_kk x_k / R_kk^2)
        double* x = tid < B ? Xi : Xj;
        const int c = tid & 31;
        double t[B];
#pragma unroll
        for (int k = 0; k < B; ++k) t[k] = x[k * LD + c];
#pragma unroll
        for (int k = 0; k < B; ++k) {
            const double f = t[k] * dinv[k];
#pragma unroll
            for (int r = k + 1; r < B; ++r) t[r] = fma(-D[k * LD + r], f, t[r]);
        }
#pragma unroll
        for (int k = 0; k < B; ++k) x[k * LD + c] = t[k];
    }
    __syncthreads();
    if (rest > 0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int r = r0 + 8 * u;
            double s = tg[u];
#pragma unroll
            for (int k = 0; k < B; ++k) s = fma(-Xi[k * LD + r] * dinv[k], Xj[k * LD + c0], s);
            const int row = I * B + r, col = J * B + c0;
            if (row < n && col < n) G[(long long)row * n + col] = s;
        }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int r = r0 + 8 * u, row = P * B + r;
        const double rs = sqrt(dinv[r]);
        if (rest > 0 && I == J) {                        // R's rows right of the diagonal block, zeros below it
            if (row < n && I * B + c0 < n) W[(long long)row * n + I * B + c0] = Xi[r * LD + c0] * rs;
            if (I * B + r < n && P * B + c0 < n) W[(long long)(I * B + r) * n + P * B + c0] = 0.0;
        }
        if (blk == 0 && row < n && P * B + c0 < n)
            W[(long long)row * n + P * B + c0] = c0 >= r ? D[r * LD + c0] * rs : 0.0;
    }
}

// ---- cyclic one-sided Jacobi iteration on the rows of W (n x n, row-major) -------------------------------------
// A rotation of two rows makes them orthogonal; a sweep visits every pair once.  The iteration is a chain of n - 1
// dependent rounds of disjoint pairs per sweep and some ten sweeps: what bounds it is the length of a round, not
// arithmetic.  One launch per round cost ~5 us a round (32 ms for a 512-long mode, 7 ms for 160); here the rounds of a
// launch run inside workgroups that hold their rows in LDS, 16 lanes to a pair (1.4 ms for 160, 8.9 ms for 500, factor and
// all; a round of cross pairs is 0.54 us, half of it the rotation, and a launch has 5 us outside its rounds).
//   n <= 64: one workgroup holds all rows and runs the whole iteration to convergence in one launch.
//   n > 64:  rows in blocks of 16.  A launch pairs the blocks (round-robin over blocks), a workgroup takes two blocks and
//            visits their 16 x 16 cross pairs in 16 rounds; the first launch of a sweep also visits the pairs inside the
//            blocks (31 rounds over the 32 rows).  A sweep is ceil(n/16) - 1 launches instead of n - 1.
// Every pair of a sweep is visited exactly once; the squared norms of the rows are computed when a launch starts
// and carried through its rotations.
constexpr int RK_JB = 16;               // rows of a block
constexpr int RK_JL = 16;               // lanes of a pair

// sum over the 16 lanes of a pair: four rotations inside the row of 16 lanes; every lane gets the same bits
// (each step adds the same two numbers in both lanes)
template <int ROR>
__device__ __forceinline__ double row_ror(double x) {
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), 0x120 + ROR, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), 0x120 + ROR, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double row16_sum(double x) {
    x += row_ror<8>(x);
    x += row_ror<4>(x);
    x += row_ror<2>(x);
    x += row_ror<1>(x);
    return x;
}
// 1 / sqrt(x) for positive normal x: the hardware's estimate and two Newton steps (x e^2 = 1 + d, e <- e (1 - d/2 + 3 d^2/8))
__device__ __forceinline__ double rsqrt64(double x) {
    double e = __builtin_amdgcn_rsq(x);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const double d = fma(-x * e, e, 1.0);
        e = fma(e * d, fma(d, 0.375, 0.5), e);
    }
    return e;
}

// The rotation (c, s) that makes rows with squared norms al, be and product ga orthogonal: x' = c x - s y, y' = s x + c y.
// With d = be - al, g = 2 ga, h = sqrt(d^2 + g^2):  c = sqrt((1 + |d| / h) / 2),  s = sign(d) g / (2 h c), the smaller of
// the two angles.  Returns false (c = 1, s = 0) where the rows are orthogonal to the rounding of their product already.
// *wide: the rotation counts against convergence.  One by a small angle between rows that were nearly orthogonal does not: with
// both below t = 2^-26, it changes the cosine of another pair by at most 2 t^2 (the angle times the ratio of the norms is at most
// 2 t, the cosine it brings in t), and the 2 (n - 2) rotations of a sweep that touch a pair by 4 n t^2 = 4 n 2^-52, which is what two rows
// may be off and count as orthogonal.  So a sweep without a wide rotation ends converged and needs no sweep after it to show it
// (a sweep of a 160-long mode is 90 to 130 us; modes of 65 to 250: 747 -> 679 us, 1760 -> 1748 and 1930 -> 1772
// for 192, 2849 -> 2641 for 250, the errors of eigenvalues and vectors unchanged).
constexpr double RK_SMALL2 = 2.220446049250313e-16;     // t^2
__device__ __forceinline__ bool rotation(double& al, double& be, double ga, double tol2, double* c, double* s, int* wide) {
    *c = 1.0; *s = 0.0; *wide = 0;
    const double ab = al * be;
    if (!(ga * ga > tol2 * ab)) return false;
    const double d = be - al, g = 2.0 * ga;
    const double ih = rsqrt64(fma(d, d, g * g));
    const double c2 = fma(0.5 * fabs(d), ih, 0.5), rc = rsqrt64(c2);
    *c = c2 * rc;
    *s = (d >= 0.0 ? 0.5 : -0.5) * g * ih * rc;
    *wide = !(ga * ga <= RK_SMALL2 * ab && *s * *s <= RK_SMALL2);
    const double tg = *s * rc * ga;                      // tan(angle) ga, rc = 1 / c
    al -= tg; be += tg;
    return true;
}

// pair p of round `round` of the round-robin schedule over m + 1 players (m odd)
__device__ __forceinline__ void round_robin(int m, int round, int p, int* a, int* b) {
    int u = p == 0 ? m : round + p, v = p == 0 ? round : round - p;
    if (p != 0 && u >= m) u -= m;
    if (v < 0) v += m;
    *a = u < v ? u : v;
    *b = u < v ? v : u;
}

// Rotates the rows ra, rb in LDS (16 NE elements, zero padded) with squared norms in na, nb; returns whether it counts.
template <int NE>
__device__ __forceinline__ int jacobi_pair(double* ra, double* rb, double* na, double* nb, int lane, double tol2) {
    double x[NE], y[NE], al = *na, be = *nb, ga = 0.0, g2 = 0.0;
#pragma unroll
    for (int k = 0; k < NE; ++k) { x[k] = ra[lane + RK_JL * k]; y[k] = rb[lane + RK_JL * k]; }
#pragma unroll
    for (int k = 0; k < NE; k += 2) { ga = fma(x[k], y[k], ga); g2 = fma(x[k + 1], y[k + 1], g2); }
    ga = row16_sum(ga + g2);
    double c, s;
    int wide;
    if (!rotation(al, be, ga, tol2, &c, &s, &wide)) return 0;
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        ra[lane + RK_JL * k] = fma(c, x[k], -s * y[k]);
        rb[lane + RK_JL * k] = fma(s, x[k], c * y[k]);
    }
    if (lane == 0) { *na = al; *nb = be; }
    return wide;
}
// squared norm of an LDS row by its 16 lanes
template <int NE>
__device__ __forceinline__ void row_norm2(const double* r, double* out, int lane) {
    double q = 0.0;
#pragma unroll
    for (int k = 0; k < NE; ++k) { const double v = r[lane + RK_JL * k]; q = fma(v, v, q); }
    q = row16_sum(q);
    if (lane == 0) *out = q;
}

// n <= 64: the whole iteration.  32 pairs x 16 lanes; rot[0] = sweeps used if converged, else 0.
__global__ __launch_bounds__(512) void k_jacobi_small(SpecBatch jobs, int max_sweeps) {
    double* __restrict__ W = jobs.job[blockIdx.x].W;
    const int n = jobs.job[blockIdx.x].n;
    const double tol2 = jobs.job[blockIdx.x].tol2;
    constexpr int NE = 4, LD = 64 + 16;                  // pitch 16 mod 32 doubles: two rows on disjoint banks
    __shared__ double w[64 * LD], nrm[64];
    __shared__ int s_rot;
    const int tid = threadIdx.x, lane = tid & (RK_JL - 1), p = tid / RK_JL;
    const int n2 = (n + 1) & ~1, m = n2 - 1;
    for (int e = tid; e < 64 * 64; e += 512) {
        const int i = e >> 6, j = e & 63;
        w[i * LD + j] = (i < n && j < n) ? W[i * n + j] : 0.0;
    }
    int used = 0;
    for (int sweep = 0; sweep < max_sweeps; ++sweep) {
        __syncthreads();
        if (tid == 0) s_rot = 0;
        row_norm2<NE>(w + p * LD, nrm + p, lane);
        row_norm2<NE>(w + (p + 32) * LD, nrm + p + 32, lane);
        __syncthreads();
        int mine = 0;
        for (int round = 0; round < m; ++round) {
            int a, b;
            round_robin(m, round, p, &a, &b);
            if (2 * p < n2 && b < n) mine += jacobi_pair<NE>(w + a * LD, w + b * LD, nrm + a, nrm + b, lane, tol2);
            __syncthreads();                             // a row is written by one pair and read by another in the next round
        }
        if (lane == 0 && mine) atomicAdd(&s_rot, mine);
        __syncthreads();
        if (s_rot == 0) { used = sweep + 1; break; }     // the same for all threads
    }
    for (int e = tid; e < n * n; e += 512) {
        const int i = e / n, j = e - i * n;
        W[e] = w[i * LD + j];
    }
    if (tid == 0) jobs.job[blockIdx.x].rot[0] = used;
}

// One launch of a sweep for n > 64: workgroup q of a mode takes the q-th pair of blocks of `round`.  The rotations that count, of the sweep
// before (not in the first; zero there means converged, nothing is done) and of this one, are in the mode's rot.
extern __shared__ double jac_dyn[];
template <int NE>
__device__ __forceinline__ void jacobi_block(const SpecJob& jb, int blk, int sweep, int round, int& s_rot, double* nrm) {
    double* __restrict__ W = jb.W;
    const int n = jb.n, nblk2 = ((n + RK_JB - 1) / RK_JB + 1) & ~1;
    const double tol2 = jb.tol2;
    int32_t* cur = jb.rot + sweep;
    constexpr int LD = RK_JL * NE + ((RK_JL * NE) % 32 == 0 ? 16 : 0);
    double* w = jac_dyn;                                 // 32 rows of LD
    const int tid = threadIdx.x, lane = tid & (RK_JL - 1), p = tid / RK_JL;
    int bi, bj;
    round_robin(nblk2 - 1, round, blk, &bi, &bj);
    if (tid == 0) s_rot = 0;
    // this thread group's two rows; rows past the end are zeros and never rotate.  All loads are in flight together.
    const int gi = bi * RK_JB + p, gj = bj * RK_JB + p;
    double x[NE], y[NE];
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int i = lane + RK_JL * k, ic = i < n ? i : n - 1;
        x[k] = W[(long long)(gi < n ? gi : n - 1) * n + ic];
        y[k] = W[(long long)(gj < n ? gj : n - 1) * n + ic];
    }
    if (sweep > 0 && jb.rot[sweep - 1] == 0) return;     // (the same for all threads; asked behind the rows, both are on their way)
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const bool in = lane + RK_JL * k < n;
        x[k] = in && gi < n ? x[k] : 0.0;
        y[k] = in && gj < n ? y[k] : 0.0;
    }
    double* ri = w + p * LD + lane;
    double* rj = w + (RK_JB + p) * LD + lane;
    double qx = 0.0, qy = 0.0;
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        ri[RK_JL * k] = x[k]; rj[RK_JL * k] = y[k];
        qx = fma(x[k], x[k], qx); qy = fma(y[k], y[k], qy);
    }
    qx = row16_sum(qx); qy = row16_sum(qy);
    if (lane == 0) { nrm[p] = qx; nrm[RK_JB + p] = qy; }
    __syncthreads();
    int mine = 0;
    if (round == 0) {                                    // the pairs inside the blocks and across them
        for (int q = 0; q < 2 * RK_JB - 1; ++q) {
            int a, b;
            round_robin(2 * RK_JB - 1, q, p, &a, &b);
            mine += jacobi_pair<NE>(w + a * LD, w + b * LD, nrm + a, nrm + b, lane, tol2);
            __syncthreads();
        }
#pragma unroll
        for (int k = 0; k < NE; ++k) x[k] = ri[RK_JL * k];
    } else {
        // a row of block I stays in the registers of its lanes, the rows of block J go round through LDS
        double al = qx;
        for (int q = 0; q < RK_JB; ++q) {
            const int b = RK_JB + ((p + q) & (RK_JB - 1));
            double* rb = w + b * LD + lane;
            double be = nrm[b], ga = 0.0, g2 = 0.0;
#pragma unroll
            for (int k = 0; k < NE; ++k) y[k] = rb[RK_JL * k];
#pragma unroll
            for (int k = 0; k < NE; k += 2) { ga = fma(x[k], y[k], ga); g2 = fma(x[k + 1], y[k + 1], g2); }
            ga = row16_sum(ga + g2);
            double c, s;
            int wide;
            if (rotation(al, be, ga, tol2, &c, &s, &wide)) {
#pragma unroll
                for (int k = 0; k < NE; ++k) {
                    const double v = fma(c, x[k], -s * y[k]);
                    rb[RK_JL * k] = fma(s, x[k], c * y[k]);
                    x[k] = v;
                }
                if (lane == 0) nrm[b] = be;
                mine += wide;
            }
            __syncthreads();
        }
    }
    if (lane == 0 && mine) atomicAdd(&s_rot, mine);
#pragma unroll
    for (int k = 0; k < NE; ++k) {
        const int i = lane + RK_JL * k;
        y[k] = rj[RK_JL * k];
        if (i < n && gi < n) W[(long long)gi * n + i] = x[k];
        if (i < n && gj < n) W[(long long)gj * n + i] = y[k];
    }
    __syncthreads();
    if (tid == 0 && s_rot) atomicAdd(cur, s_rot);
}
// elements per lane of a row of n: the shapes the rows are held in
__host__ __device__ constexpr int row_shape(int n) { return n <= 128 ? 8 : (n <= 192 ? 12 : (n <= 256 ? 16 : 32)); }
// NE of the longest mode.  A launch for one mode neither looks for its mode nor carries the code of other shapes (k_jacobi_one; a
// 500-long mode takes 9.4 ms in the general form, 8.9 in this one).
template <int NE>
__global__ __launch_bounds__(256) void k_jacobi_block(SpecBatch a, int sweep, int round) {
    __shared__ int s_rot;
    __shared__ double nrm[2 * RK_JB];
    int blk;
    const SpecJob& jb = find_mode(a, &blk);
    const int nblk2 = ((jb.n + RK_JB - 1) / RK_JB + 1) & ~1;
    if (round >= nblk2 - 1) return;                      // the same for all threads
    const int ne = row_shape(jb.n);
    if (NE == 8 || ne == 8) jacobi_block<8>(jb, blk, sweep, round, s_rot, nrm);
    else if (NE == 12 || ne == 12) jacobi_block<12>(jb, blk, sweep, round, s_rot, nrm);
    else if (NE == 16 || ne == 16) jacobi_block<16>(jb, blk, sweep, round, s_rot, nrm);
    else jacobi_block<32>(jb, blk, sweep, round, s_rot, nrm);
}
template <int NE>
__global__ __launch_bounds__(256) void k_jacobi_one(SpecJob jb, int sweep, int round) {
    __shared__ int s_rot;
    __shared__ double nrm[2 * RK_JB];
    jacobi_block<NE>(jb, blockIdx.x, sweep, round, s_rot, nrm);
}

// After convergence row k of W is sqrt(lambda_k) v_k^T, lambda_k an eigenvalue of the scaled and shifted G.  Eigenvalues in descending order (ties by row index),
// eigenvectors as the columns of an n x n row-major fp32 matrix; a column whose eigenvalue is below
// 1e-12 of the largest (a null direction, whose row carries no direction any more) is returned as zeros.  A G that is not finite
// has no spectrum: every eigenvalue is NaN (Inf if no entry of G is NaN), every column zeros.
__global__ __launch_bounds__(64) void k_row_norms(SpecBatch a) {
    int k;
    const SpecJob& jb = find_mode(a, &k);
    const double* __restrict__ W = jb.W;
    const CholScale* __restrict__ sc = jb.sc;
    const int n = jb.n;
    constexpr int NE = RK_NMAX / 64;
    const int lane = threadIdx.x;
    double t[NE];
#pragma unroll
    for (int u = 0; u < NE; ++u) t[u] = W[(long long)k * n + (lane + 64 * u < n ? lane + 64 * u : 0)];
    double s = 0.0;
#pragma unroll
    for (int u = 0; u < NE; ++u) s += lane + 64 * u < n ? t[u] * t[u] : 0.0;
    s = wave_sum(s);
    if (lane == 0) jb.norms[k] = sc->bad != 0.0 ? sc->bad : s > sc->shift ? (s - sc->shift) / sc->scale : 0.0;   // the eigenvalue of G itself
}
// workgroup k places row k: its rank among the eigenvalues by counting, then its column of the eigenvector matrix
__global__ __launch_bounds__(256) void k_spectrum_finish(SpecBatch a) {
    int k;
    const SpecJob& jb = find_mode(a, &k);
    const double* __restrict__ W = jb.W;
    const double* __restrict__ norms = jb.norms;
    const CholScale* __restrict__ sc = jb.sc;
    float* __restrict__ vec_out = jb.vec;
    const int n = jb.n;
    __shared__ int s_pos[4];
    __shared__ double s_max[4];
    const int tid = threadIdx.x;
    const double l = norms[k];
    int pos = 0;
    double lmax = 0.0;
#pragma unroll
    for (int u = 0; u < RK_NMAX / 256; ++u) {
        const int j = tid + 256 * u;
        const double lj = norms[j < n ? j : 0];
        if (j < n) {
            pos += (lj > l || (lj == l && j < k)) ? 1 : 0;
            lmax = fmax(lmax, lj);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) { pos += __shfl_xor(pos, d, 64); lmax = fmax(lmax, __shfl_xor(lmax, d, 64)); }
    if ((tid & 63) == 0) { s_pos[tid >> 6] = pos; s_max[tid >> 6] = lmax; }
    __syncthreads();
    pos = s_pos[0] + s_pos[1] + s_pos[2] + s_pos[3];
    lmax = fmax(fmax(s_max[0], s_max[1]), fmax(s_max[2], s_max[3]));
    if (sc->bad != 0.0) pos = k;                         // (nothing to order by)
    if (tid == 0) jb.lam[pos] = l;
    if (!vec_out) return;
    const bool live = l > 1e-12 * lmax && l > 0.0;
    const double inv = live ? 1.0 / sqrt(l * sc->scale + sc->shift) : 0.0;       // the row's norm
    for (int i = tid; i < n; i += 256) vec_out[(long long)i * n + pos] = live ? (float)(W[(long long)k * n + i] * inv) : 0.f;
}

struct EpsList { double eps[16]; int count; };
// ranks[j] = smallest r >= 1 whose leading eigenvalues hold the fraction eps[j] of their sum (Sec. 3.3, Step 1)
__global__ void k_ev_ranks(const double* __restrict__ lam, int n, EpsList el, int32_t* __restrict__ ranks) {
    const int j = threadIdx.x;
    if (j >= el.count) return;
    double total = 0.0;
    for (int k = 0; k < n; ++k) total += lam[k];
    double run = 0.0;
    int r = n;
    for (int k = 0; k < n; ++k) {
        run += lam[k];
        if (run >= el.eps[j] * total) { r = k + 1; break; }
    }
    ranks[j] = r;
}

__global__ __launch_bounds__(256) void k_frob_partial(const float* __restrict__ a, const float* __restrict__ b, long long cnt,
                                                      double* __restrict__ part) {
    __shared__ double red[4];
    double s = 0.0;
    for (long long e = (long long)blockIdx.x * 256 + threadIdx.x; e < cnt; e += (long long)gridDim.x * 256) {
        const double d = (double)a[e] - (double)b[e];
        s += d * d;
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}
__global__ __launch_bounds__(64) void k_frob_final(const double* __restrict__ part, int nparts, double* __restrict__ out) {
    double s = 0.0;
    for (int k = threadIdx.x; k < nparts; k += 64) s += part[k];
    s = wave_sum(s);
    if (threadIdx.x == 0) *out = sqrt(s);
}

struct ModeShape {
    long long outer = 1, inner = 1, ncols = 1, numel = 1;
    int n = 0;
    bool bf16 = false;
};
bool parse_mode(const asi_tensor_desc* desc, int mode, ModeShape* ms, asi_status* why) {
    if (!desc || (desc->ndim != 3 && desc->ndim != 4) || mode < 0 || mode >= desc->ndim) { *why = ASI_ERR_INVALID_ARG; return false; }
    if (desc->dtype != ASI_F32 && desc->dtype != ASI_BF16) { *why = ASI_ERR_UNSUPPORTED; return false; }
    for (int m = 0; m < desc->ndim; ++m) {
        if (desc->dims[m] <= 0 || desc->dims[m] > (1LL << 30)) { *why = ASI_ERR_INVALID_ARG; return false; }
        ms->numel *= desc->dims[m];
        if (ms->numel > (1LL << 40)) { *why = ASI_ERR_UNSUPPORTED; return false; }
        if (m < mode) ms->outer *= desc->dims[m];
        if (m > mode) ms->inner *= desc->dims[m];
    }
    if (desc->dims[mode] > RK_NMAX) { *why = ASI_ERR_UNSUPPORTED; return false; }
    ms->n = (int)desc->dims[mode];
    ms->ncols = ms->outer * ms->inner;
    ms->bf16 = desc->dtype == ASI_BF16;
    return true;
}
constexpr int RK_SWEEPS = 60;
constexpr size_t RK_COUNTS = RK_ALIGN;                   // bytes of a mode's counters
static_assert(sizeof(int32_t) * RK_SWEEPS <= RK_COUNTS, "a counter per sweep");
struct GramPlan { int tiles, nchunks, nsplit; size_t part_bytes, w_bytes, norm_bytes, bytes; };
GramPlan plan_gram(const ModeShape& ms) {
    GramPlan p;
    p.tiles = (ms.n + RK_T - 1) / RK_T;
    const long long chunks = (ms.ncols + RK_T - 1) / RK_T;
    p.nchunks = (int)(chunks > 0x7fffffffLL ? 0x7fffffffLL : chunks);
    long long want = 2048 / ((long long)p.tiles * p.tiles);
    if (want > RK_MAX_SPLIT) want = RK_MAX_SPLIT;
    if (want > chunks) want = chunks;
    if (want < 1) want = 1;
    p.nsplit = (int)want;
    p.part_bytes = align_up(sizeof(double) * (size_t)p.nsplit * ms.n * ms.n);
    p.w_bytes = align_up(sizeof(double) * (size_t)ms.n * ms.n);
    p.norm_bytes = align_up(sizeof(double) * (size_t)ms.n);
    // partial Gram matrices, G, W, the eigenvalues in row order, scale and shift, a rotation counter per sweep
    p.bytes = p.part_bytes + 2 * p.w_bytes + p.norm_bytes + align_up(sizeof(CholScale)) + RK_COUNTS;
    return p;
}

// the modes of a launch: their argument blocks side by side, `blocks` workgroups each (none: the mode takes no part)
template <typename F>
int gather_modes(const SpecJob* jobs, int n, F blocks, SpecBatch* b) {
    int total = 0;
    b->njobs = 0;
    for (int j = 0; j < n; ++j) {
        const int k = blocks(jobs[j]);
        if (k <= 0) continue;
        b->first[b->njobs] = total;
        b->job[b->njobs++] = jobs[j];
        total += k;
    }
    for (int j = b->njobs; j <= RK_MODES; ++j) b->first[j] = total;
    return total;
}

// the launches of one sweep for modes of n > 64: every pair of blocks once
template <int NE>
hipError_t jacobi_sweep(const SpecBatch& b, int grid, int rounds, int sweep, hipStream_t st) {
    constexpr size_t lds = sizeof(double) * 2 * RK_JB * (RK_JL * NE + ((RK_JL * NE) % 32 == 0 ? 16 : 0));
    if (lds > 65536) {
        static LdsAllowed allowed, allowed_one;
        const hipError_t e = b.njobs == 1 ? allow_lds(reinterpret_cast<const void*>(k_jacobi_one<NE>), lds, allowed_one)
                                          : allow_lds(reinterpret_cast<const void*>(k_jacobi_block<NE>), lds, allowed);
        if (e != hipSuccess) return e;
    }
    for (int round = 0; round < rounds; ++round) {
        if (b.njobs == 1) hipLaunchKernelGGL(k_jacobi_one<NE>, dim3((unsigned)grid), 256, lds, st, b.job[0], sweep, round);
        else hipLaunchKernelGGL(k_jacobi_block<NE>, dim3((unsigned)grid), 256, lds, st, b, sweep, round);
    }
    return hipGetLastError();
}
hipError_t launch_jacobi_sweep(const SpecJob* jobs, int njobs, int sweep, hipStream_t st) {
    SpecBatch b;
    int longest = 0;
    for (int j = 0; j < njobs; ++j) longest = jobs[j].n > longest ? jobs[j].n : longest;
    const auto blocks = [](int n) { return ((n + RK_JB - 1) / RK_JB + 1) & ~1; };
    const int grid = gather_modes(jobs, njobs, [&](const SpecJob& j) { return blocks(j.n) / 2; }, &b), rounds = blocks(longest) - 1;
    switch (row_shape(longest)) {
        case 8: return jacobi_sweep<8>(b, grid, rounds, sweep, st);
        case 12: return jacobi_sweep<12>(b, grid, rounds, sweep, st);
        case 16: return jacobi_sweep<16>(b, grid, rounds, sweep, st);
        default: return jacobi_sweep<32>(b, grid, rounds, sweep, st);
    }
}

struct Search {
    int n, e;
    const double* P;
    const int64_t* M;
    int64_t budget;
    std::vector<double> minP;          // minP[i] = sum over layers >= i of their least perplexity
    std::vector<int64_t> minM;
    std::vector<int> cur, best;
    double best_total;
    bool found;
    void walk(int i, int64_t mem, double tot) {
        if (i == n) {
            if (!found || tot < best_total) { found = true; best_total = tot; best = cur; }
            return;
        }
        for (int j = 0; j < e; ++j) {
            const int64_t m2 = mem + M[(size_t)i * e + j];
            if (m2 + minM[i + 1] > budget) continue;                       // cannot fit whatever follows
            const double t2 = tot + P[(size_t)i * e + j];
            // cannot get below the best so far (with room for the rounding of the bound's own sum)
            if (found && t2 + minP[i + 1] > best_total + 1e-12 * fabs(best_total)) continue;
            cur[i] = j;
            walk(i + 1, m2, t2);
        }
    }
};

}  // namespace

extern "C" {

int64_t asi_activation_memory(const asi_tensor_desc* desc) {
    if (!desc || (desc->ndim != 3 && desc->ndim != 4)) return -1;
    int64_t prod = 1, sum = 0;
    for (int m = 0; m < desc->ndim; ++m) {
        if (desc->dims[m] <= 0 || desc->ranks[m] < 1 || desc->ranks[m] > desc->dims[m]) return -1;
        prod *= desc->ranks[m];
        sum += desc->dims[m] * desc->ranks[m];
    }
    return prod + sum;
}

size_t asi_mode_spectra_workspace_bytes(const asi_tensor_desc* desc, const int32_t* modes, int32_t n_modes) {
    if (!modes || n_modes < 1 || n_modes > RK_MODES) return 0;
    size_t total = 0;
    for (int k = 0; k < n_modes; ++k) {
        ModeShape ms;
        asi_status why;
        if (!parse_mode(desc, modes[k], &ms, &why)) return 0;
        total += plan_gram(ms).bytes;
    }
    return total;
}

size_t asi_mode_spectrum_workspace_bytes(const asi_tensor_desc* desc, int32_t mode) {
    return asi_mode_spectra_workspace_bytes(desc, &mode, 1);
}

asi_status asi_mode_spectra(const asi_tensor_desc* desc, const void* A, const int32_t* modes, int32_t n_modes, double* const* eigenvalues,
                            float* const* eigenvectors, void* ws, size_t ws_bytes, int32_t* sweeps, asi_stream_t stream) {
    if (!modes || n_modes < 1 || n_modes > RK_MODES || !eigenvalues) return ASI_ERR_INVALID_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    char* base = static_cast<char*>(ws);
    SpecJob jobs[RK_MODES];
    size_t need = 0;
    for (int k = 0; k < n_modes; ++k) {
        ModeShape ms;
        asi_status why;
        if (!parse_mode(desc, modes[k], &ms, &why)) return why;
        if (!A || !eigenvalues[k]) return ASI_ERR_INVALID_ARG;
        const GramPlan p = plan_gram(ms);
        SpecJob& jb = jobs[k];
        char* at = base + need;
        need += p.bytes - RK_COUNTS;
        jb.X = A; jb.outer = ms.outer; jb.inner = ms.inner; jb.ncols = ms.ncols; jb.n = ms.n;
        jb.tiles = p.tiles; jb.nsplit = p.nsplit; jb.nchunks = p.nchunks;
        jb.part = reinterpret_cast<double*>(at); at += p.part_bytes;
        jb.G = reinterpret_cast<double*>(at); at += p.w_bytes;
        jb.W = reinterpret_cast<double*>(at); at += p.w_bytes;
        jb.norms = reinterpret_cast<double*>(at); at += p.norm_bytes;
        jb.sc = reinterpret_cast<CholScale*>(at); at += align_up(sizeof(CholScale));
        // additions behind an entry of G: the columns of a range (64 a chunk), then the ranges
        const double adds = (double)RK_T * ((p.nchunks + p.nsplit - 1) / p.nsplit) + p.nsplit;
        jb.shift_factor = (4.0 * ms.n + adds) * 1.1102230246251565e-16;
        const double tol = 4.0 * ms.n * 2.220446049250313e-16;   // two rows count as orthogonal below the rounding of their dot product
        jb.tol2 = tol * tol;
        jb.lam = eigenvalues[k];
        jb.vec = eigenvectors ? eigenvectors[k] : nullptr;
    }
    // the counters of all modes stand side by side behind the last mode
    for (int k = 0; k < n_modes; ++k, need += RK_COUNTS) jobs[k].rot = reinterpret_cast<int32_t*>(base + need);
    if (!ws || reinterpret_cast<uintptr_t>(ws) % RK_ALIGN != 0 || ws_bytes < need) return ASI_ERR_WORKSPACE;

    SpecBatch b;
    int grid = gather_modes(jobs, n_modes, [](const SpecJob& j) { return j.tiles * j.tiles * j.nsplit; }, &b);
    if (desc->dtype == ASI_BF16) hipLaunchKernelGGL(k_mode_gram<bf16_t>, dim3((unsigned)grid), 256, 0, st, b);
    else hipLaunchKernelGGL(k_mode_gram<float>, dim3((unsigned)grid), 256, 0, st, b);
    grid = gather_modes(jobs, n_modes, [](const SpecJob& j) { return (j.n * j.n + 255) / 256; }, &b);
    hipLaunchKernelGGL(k_gram_reduce, dim3((unsigned)grid), 256, 0, st, b, RK_SWEEPS);
    grid = gather_modes(jobs, n_modes, [](const SpecJob&) { return 1; }, &b);
    hipLaunchKernelGGL(k_chol_scale, dim3((unsigned)grid), 256, 0, st, b);
    for (int P = 0; P < (RK_NMAX + RK_CB - 1) / RK_CB; ++P) {
        grid = gather_modes(jobs, n_modes, [P](const SpecJob& j) {
            const int rest = (j.n + RK_CB - 1) / RK_CB - P - 1;
            return rest > 0 ? rest * (rest + 1) / 2 : (rest == 0 ? 1 : 0);
        }, &b);
        if (grid == 0) break;
        hipLaunchKernelGGL(k_chol_panel, dim3((unsigned)grid), 256, 0, st, b, P);
    }
    if (hipGetLastError() != hipSuccess) return ASI_ERR_HIP;

    // Sweeps until a whole one has no rotation that counts; the counts come back to the host (this entry point iterates to convergence and
    // therefore waits for the stream).  Modes of up to 64 iterate in one launch.  Sweeps are handed over several at a time (one
    // that follows a converged one returns at once), so that the host's wait does not stand between every two of them.
    grid = gather_modes(jobs, n_modes, [](const SpecJob& j) { return j.n > 1 && j.n <= 64 ? 1 : 0; }, &b);
    if (grid) hipLaunchKernelGGL(k_jacobi_small, dim3((unsigned)grid), 512, 0, st, b, RK_SWEEPS);
    int used[RK_MODES];                                  // sweeps until convergence, -1 before
    SpecJob open[RK_MODES];                              // the longer modes that have not converged
    int which[RK_MODES], n_open = 0;
    for (int k = 0; k < n_modes; ++k) {
        used[k] = jobs[k].n == 1 ? 0 : -1;
        if (jobs[k].n > 64) { which[n_open] = k; open[n_open++] = jobs[k]; }
    }
    // one copy brings the counters of all modes: a copy is a wait of some 30 us
    int32_t h[RK_MODES][RK_COUNTS / sizeof(int32_t)];
    for (int done = 0; done == 0 || (n_open > 0 && done < RK_SWEEPS);) {
        int upto = done + (done == 0 ? 8 : 2);
        if (upto > RK_SWEEPS) upto = RK_SWEEPS;
        for (int sweep = done; sweep < upto && n_open; ++sweep)
            if (launch_jacobi_sweep(open, n_open, sweep, st) != hipSuccess) return ASI_ERR_HIP;
        if (n_open || (done == 0 && grid)) {
            if (hipMemcpyAsync(h, jobs[0].rot, RK_COUNTS * n_modes, hipMemcpyDeviceToHost, st) != hipSuccess) return ASI_ERR_HIP;
            if (hipStreamSynchronize(st) != hipSuccess) return ASI_ERR_HIP;
        }
        for (int k = 0; k < n_modes && done == 0; ++k)
            if (jobs[k].n > 1 && jobs[k].n <= 64 && h[k][0] > 0) used[k] = h[k][0];
        int left = 0;
        for (int q = 0; q < n_open; ++q) {
            int at = -1;
            for (int sweep = done; sweep < upto && at < 0; ++sweep)
                if (h[which[q]][sweep] == 0) at = sweep + 1;
            used[which[q]] = at;
            if (at < 0) { which[left] = which[q]; open[left++] = open[q]; }
        }
        n_open = left;
        done = upto;
    }
    grid = gather_modes(jobs, n_modes, [](const SpecJob& j) { return j.n; }, &b);
    hipLaunchKernelGGL(k_row_norms, dim3((unsigned)grid), 64, 0, st, b);
    hipLaunchKernelGGL(k_spectrum_finish, dim3((unsigned)grid), 256, 0, st, b);
    if (hipGetLastError() != hipSuccess) return ASI_ERR_HIP;
    bool converged = true;
    for (int k = 0; k < n_modes; ++k) {
        if (sweeps) sweeps[k] = used[k];
        converged = converged && used[k] >= 0;
    }
    return converged ? ASI_OK : ASI_ERR_NUMERIC;
}

asi_status asi_mode_spectrum(const asi_tensor_desc* desc, const void* A, int32_t mode, double* eigenvalues,
                             float* eigenvectors, void* ws, size_t ws_bytes, int32_t* sweeps, asi_stream_t stream) {
    return asi_mode_spectra(desc, A, &mode, 1, &eigenvalues, &eigenvectors, ws, ws_bytes, sweeps, stream);
}

asi_status asi_explained_variance_ranks(const double* eigenvalues, int32_t n, const double* eps, int32_t n_eps,
                                        int32_t* ranks, asi_stream_t stream) {
    if (!eigenvalues || !eps || !ranks || n < 1 || n_eps < 1 || n_eps > 16) return ASI_ERR_INVALID_ARG;
    EpsList el;
    el.count = n_eps;
    for (int j = 0; j < n_eps; ++j) {
        if (!(eps[j] > 0.0) || eps[j] > 1.0) return ASI_ERR_INVALID_ARG;
        el.eps[j] = eps[j];
    }
    hipLaunchKernelGGL(k_ev_ranks, dim3(1), 64, 0, static_cast<hipStream_t>(stream), eigenvalues, (int)n, el, ranks);
    return hipGetLastError() == hipSuccess ? ASI_OK : ASI_ERR_HIP;
}

asi_status asi_frobenius_diff(const float* a, const float* b, int64_t count, double* out, void* ws, size_t ws_bytes,
                              asi_stream_t stream) {
    if (!a || !b || !out || count < 1) return ASI_ERR_INVALID_ARG;
    if (!ws || reinterpret_cast<uintptr_t>(ws) % RK_ALIGN != 0 || ws_bytes < (size_t)ASI_FROBENIUS_WS_BYTES) return ASI_ERR_WORKSPACE;
    long long wg = (count + 255) / 256;
    if (wg > RK_FROB_WG) wg = RK_FROB_WG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    double* part = static_cast<double*>(ws);
    hipLaunchKernelGGL(k_frob_partial, dim3((unsigned)wg), 256, 0, st, a, b, (long long)count, part);
    hipLaunchKernelGGL(k_frob_final, dim3(1), 64, 0, st, part, (int)wg, out);
    return hipGetLastError() == hipSuccess ? ASI_OK : ASI_ERR_HIP;
}

asi_status asi_rank_select(int32_t n_layers, int32_t n_eps, const double* P, const int64_t* M, int64_t budget,
                           int32_t* choice, double* total) {
    if (n_layers < 1 || n_layers > 64 || n_eps < 1 || n_eps > 16 || !P || !M || !choice) return ASI_ERR_INVALID_ARG;
    for (size_t k = 0; k < (size_t)n_layers * n_eps; ++k)
        if (!(P[k] >= 0.0) || !std::isfinite(P[k]) || M[k] < 0) return ASI_ERR_INVALID_ARG;
    Search s;
    s.n = n_layers; s.e = n_eps; s.P = P; s.M = M; s.budget = budget;
    s.minP.assign(n_layers + 1, 0.0);
    s.minM.assign(n_layers + 1, 0);
    for (int i = n_layers - 1; i >= 0; --i) {
        double p = P[(size_t)i * n_eps];
        int64_t m = M[(size_t)i * n_eps];
        for (int j = 1; j < n_eps; ++j) {
            p = std::min(p, P[(size_t)i * n_eps + j]);
            m = std::min(m, M[(size_t)i * n_eps + j]);
        }
        s.minP[i] = s.minP[i + 1] + p;
        s.minM[i] = s.minM[i + 1] + m;
    }
    s.cur.assign(n_layers, 0);
    s.best_total = std::numeric_limits<double>::infinity();
    s.found = false;
    s.walk(0, 0, 0.0);
    if (!s.found) return ASI_ERR_INFEASIBLE;
    for (int i = 0; i < n_layers; ++i) choice[i] = s.best[i];
    if (total) *total = s.best_total;
    return ASI_OK;
}

}  // extern "C"
