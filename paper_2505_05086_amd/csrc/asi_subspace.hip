// Fused subspace-iteration step for modes with a short fibre (n <= 64) over few columns: what the Gram-matrix
// kernels (asi_gram.hip, asi_planes.hip) leave.
//
// For such a mode the two products of Alg. 1, V = A_m^T U_prev and P = A_m V, are done
// on the same LDS tile of complete mode-m fibres, so V never exists in memory and the
// activation is read once:   P = sum over fibres x of  x (x^T U_prev).
//   step A (fp32 MFMA 16x16x4):  V[c,q]  = sum_i X[i,c] U[i,q]      16 fibres at a time
//   step B (fp64 MFMA 16x16x4):  P[i,q] += sum_c X[i,c] V[c,q]      accumulators stay in registers
// The accumulator layout of step A (lane l, register v holds fibre 4*(l/16)+v, column l%16)
// is exactly the B-operand layout step B needs if step B walks the 16 fibres in the order
// k-step v -> fibres {v, 4+v, 8+v, 12+v}; the A operand is fetched from LDS in that order.
// P is summed in fp64: the columns of U_prev need not be aligned with singular vectors, so
// P holds components (sigma_r/sigma_1)^2 below its largest ones that fp32 sums would lose.
//
// A tile is a run of complete outer slices (contiguous memory).  All loads of a tile are issued
// before the first is stored (one memory latency per tile); two or more workgroups per CU overlap
// one tile's loads with another's MFMAs.  A long inner extent of 49 to 64 entries takes no tile
// (asi_subspace_cols.h).
#include "asi_device.h"
#include "asi_kernels.h"
#include "asi_subspace_cols.h"
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

constexpr int SS_TC = 128;                 // fibres (unfolding columns) per tile
constexpr int SS_PAD = 4;
constexpr int SS_LDS_FLOATS = 64 * (SS_TC + SS_PAD);   // 33 KB
constexpr int SS_PRE = (SS_LDS_FLOATS + 255) / 256;    // prefetch registers per thread
static const int SS_MAX_WG = 1024;

struct SmallView {
    const float* U;      // (n, r) previous factor
    double* part;        // (nwg, n, r) partial sums of P
    int n, r;
    int sI;              // LDS stride between consecutive mode indices
    int div, mulA, mulB; // LDS offset of fibre c at mode index 0: (c / div) * mulA + (c % div) * mulB
    float inv_div;       // 1 / div: c stays below 2^14, so the rounded float quotient is exact
    int cols_per_o;      // fibres one outer slice contributes
};
struct SmallJob {
    const void* X;
    long long outer;     // outer slices
    long long o_elems;   // elements per outer slice
    int To;              // outer slices per tile
    long long ntiles;
    int nwg;             // workgroups of this job; each walks tiles nwg apart
    int32_t* zero;       // nullable: `nzero` int32 to clear (arrival counters of the orth launches that follow)
    int nzero;
    SmallView v;
};

template <typename T, int NBM, int NBR>
__global__ __launch_bounds__(256, 2) void k_subspace_small(Batch<SmallJob> bt) {
    int lb;
    const SmallJob& jb = bt.job[locate(bt, &lb)];
    __shared__ float smem[SS_LDS_FLOATS];
    __shared__ float Us[NBM * 16][NBR * 16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lg = lane >> 4, ll = lane & 15;
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;

    // the factors: all loads first (addresses valid for every lane), then the stores; written as a loop of
    // load and store, every element paid its own round trip to memory
    {
        constexpr int PV = NBM * 16 * NBR * 16, NU = PV / 256;
        static_assert(NU * 256 == PV, "whole passes");
        float ut[NU];
        bool uok[NU];
        {
            const float* Uv = jb.v.U;
            const int nv = jb.v.n, rv = jb.v.r;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int rem = tid + 256 * u, i = rem / (NBR * 16), q = rem - i * (NBR * 16);
                uok[u] = i < nv && q < rv;
                ut[u] = Uv[uok[u] ? (long long)i * rv + q : 0LL];
            }
        }
#pragma unroll
        for (int u = 0; u < NU; ++u) (&Us[0][0])[tid + 256 * u] = uok[u] ? ut[u] : 0.f;
    }

    v4d pacc[NBM][NBR];
#pragma unroll
    for (int mb = 0; mb < NBM; ++mb)
#pragma unroll
        for (int nb = 0; nb < NBR; ++nb) pacc[mb][nb] = (v4d){0.0, 0.0, 0.0, 0.0};

    for (long long tile = lb; tile < jb.ntiles; tile += jb.nwg) {
        __syncthreads();   // everyone is done with the previous tile (and Us is written)
        // the whole tile is requested before any of it is stored: one memory latency per tile
        const long long o0 = tile * jb.To;
        const int no = (int)((jb.outer - o0 < jb.To) ? jb.outer - o0 : jb.To);
        const int count = no * (int)jb.o_elems;
        const T* src = X + o0 * jb.o_elems;
        T prw[SS_PRE];
#pragma unroll
        for (int u = 0; u < SS_PRE; ++u) {
            const int e = u * 256 + tid;
            prw[u] = src[e < count ? e : 0];          // clamped, not branched: all loads stay in flight
        }
#pragma unroll
        for (int u = 0; u < SS_PRE; ++u) {
            const int e = u * 256 + tid;
            if (e < count) smem[e] = to_f32(prw[u]);
        }
        __syncthreads();
        {
            const SmallView& sv = jb.v;
            const int n = sv.n, sI = sv.sI;
            const int valid_cols = no * sv.cols_per_o;
            // The loop body is free of branches and every group of LDS reads is issued before the
            // products that consume it, so that a fibre block pays LDS latency twice, not once per product.
            // B operands of step A do not depend on the fibre block (rows i >= n of Us are zero)
            float ub[NBM * 4][NBR];
#pragma unroll
            for (int ks = 0; ks < NBM * 4; ++ks)
#pragma unroll
                for (int nb = 0; nb < NBR; ++nb) ub[ks][nb] = Us[4 * ks + lg][16 * nb + ll];
            for (int cb = wave; cb * 16 < valid_cols; cb += 4) {
                // step A: V for 16 fibres
                const int cA = cb * 16 + ll;
                const bool okA = cA < valid_cols;
                const int qA = (int)(((float)cA + 0.5f) * sv.inv_div);
                const int ofsA = qA * sv.mulA + (cA - qA * sv.div) * sv.mulB;
                float av[NBM * 4];
#pragma unroll
                for (int ks = 0; ks < NBM * 4; ++ks) {
                    const int i = 4 * ks + lg;
                    const bool ok = okA && i < n;
                    const float x = smem[ok ? ofsA + i * sI : 0];
                    av[ks] = ok ? x : 0.f;
                }
                v4f vacc[NBR];
#pragma unroll
                for (int nb = 0; nb < NBR; ++nb) vacc[nb] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < NBM * 4; ++ks)
#pragma unroll
                    for (int nb = 0; nb < NBR; ++nb)
                        vacc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[ks], ub[ks][nb], vacc[nb], 0, 0, 0);
                // step B: P += X V over the same 16 fibres
                double a2[4][NBM];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int cB = cb * 16 + 4 * lg + v;
                    const bool okB = cB < valid_cols;
                    const int qB = (int)(((float)cB + 0.5f) * sv.inv_div);
                    const int ofsB = qB * sv.mulA + (cB - qB * sv.div) * sv.mulB;
#pragma unroll
                    for (int mb = 0; mb < NBM; ++mb) {
                        const int i = 16 * mb + ll;
                        const bool ok = okB && i < n;
                        const float x = smem[ok ? ofsB + i * sI : 0];
                        a2[v][mb] = ok ? (double)x : 0.0;
                    }
                }
#pragma unroll
                for (int v = 0; v < 4; ++v)
#pragma unroll
                    for (int mb = 0; mb < NBM; ++mb)
#pragma unroll
                        for (int nb = 0; nb < NBR; ++nb)
                            pacc[mb][nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(a2[v][mb], (double)vacc[nb][v],
                                                                                    pacc[mb][nb], 0, 0, 0);
            }
        }
    }
    // sum the four waves' accumulators through LDS, wave after wave (fixed order)
    double* red = reinterpret_cast<double*>(smem);   // (NBM*16) x (NBR*16) doubles <= 32 KB
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int mb = 0; mb < NBM; ++mb)
#pragma unroll
                for (int nb = 0; nb < NBR; ++nb)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const int i = 16 * mb + lg + 4 * v, q = 16 * nb + ll;   // fp64 MFMA result layout
                        double* p = red + i * (NBR * 16) + q;
                        *p = (w == 0) ? pacc[mb][nb][v] : *p + pacc[mb][nb][v];
                    }
        }
        __syncthreads();
    }
    const int n = jb.v.n, r = jb.v.r;
    double* out = jb.v.part + (long long)lb * n * r;
    for (int e = tid; e < n * r; e += 256) {
        const int i = e / r, q = e - i * r;
        out[e] = red[i * (NBR * 16) + q];
    }
}

template <typename T, bool VEC>
__global__ __launch_bounds__(SC_NT, VEC ? 4 : 2) void k_subspace_cols(Batch<ColsJob> bt) {
    int lb;
    const ColsJob& jb = bt.job[locate_xcd(bt, &lb)];
    subspace_cols<T, VEC>(jb, lb);
}

// ---- host side ---------------------------------------------------------------------
static bool cols_form(int n, long long inner, int r) { return n > 48 && r <= 16 && inner >= SS_TC; }
bool subspace_small_supported(long long outer, int n, long long inner, int r) {
    if (n > 64 || r > 64 || r > n) return false;
    return inner < SS_TC || subspace_gram_supported(outer, n, inner, r) || cols_form(n, inner, r);
}

// Outer slices per tile when a tile is a run of whole slices: as many as the LDS buffer holds, but
// no fewer than ~SS_MAX_WG tiles in all: the MFMA chains of a tile are latency bound, and only
// several resident workgroups per CU hide that.
static long long whole_To(long long outer, long long o_elems) {
    long long To = SS_LDS_FLOATS / o_elems;
    const long long spread = (outer + SS_MAX_WG - 1) / SS_MAX_WG;
    if (To > spread) To = spread;
    return To < 1 ? 1 : To;
}

static long long cols_blocks(long long outer, long long inner) { return outer * ((inner + 15) / 16); }

// tile geometry of one mode seen as (outer, n, inner): runs of whole outer slices
static void single_geometry(long long outer, int n, long long inner, SmallJob* jb) {
    jb->outer = outer; jb->o_elems = (long long)n * inner;
    const long long To = whole_To(outer, (long long)n * inner);
    jb->To = (int)To;
    jb->ntiles = (outer + To - 1) / To;
}

int subspace_small_nwg(long long outer, int n, long long inner, int r) {
    if (cols_form(n, inner, r)) {
        // a block per wave up to one workgroup a CU, beyond that every wave walks as many: 392 workgroups instead of 196 11.4 us
        // against 10.4 (64 x 256 x 14 x 14), 98 15.6
        const long long wgs = (cols_blocks(outer, inner) + SC_NW - 1) / SC_NW, per = (wgs + 255) / 256;
        return (int)((wgs + per - 1) / per);
    }
    SmallJob jb;
    single_geometry(outer, n, inner, &jb);
    return (int)(jb.ntiles < SS_MAX_WG ? jb.ntiles : SS_MAX_WG);
}

// key: [0] bf16, [1] VEC (columns), [2] columns, [4..6] NBM, [8..10] NBR
bool make_subspace_small(DType xt, const void* X, long long outer, int n, long long inner, const float* U, int r,
                         double* part, int nwg, int32_t* zero, int nzero, Item* out) {
    if (!subspace_small_supported(outer, n, inner, r) || !X || !U || !part || nzero < 0 || nzero > 256) return false;
    if (nwg != subspace_small_nwg(outer, n, inner, r)) return false;
    const char* tn = xt == F32 ? "float" : "asi::bf16_t";
    *out = Item();
    out->kind = IT_SMALL;
    out->nblocks = nwg;
    if (cols_form(n, inner, r)) {
        ColsJob jb;
        std::memset(&jb, 0, sizeof(jb));
        jb.X = X; jb.U = U; jb.part = part; jb.outer = outer; jb.inner = inner; jb.nblk = cols_blocks(outer, inner);
        jb.bpo = (int)((inner + 15) / 16); jb.n = n; jb.r = r; jb.nwg = nwg; jb.zero = zero; jb.nzero = zero ? nzero : 0;
        const bool vec = inner % 4 == 0 && reinterpret_cast<uintptr_t>(X) % (xt == F32 ? 16 : 8) == 0;
        out->key = (xt == BF16 ? 1u : 0u) | (vec ? 2u : 0u) | 4u;
        std::snprintf(out->label, sizeof(out->label), "k_subspace_cols<%s, %s>", tn, vec ? "true" : "false");
        static_assert(sizeof(ColsJob) <= kItemArgMax, "argument block");
        std::memcpy(out->arg, &jb, sizeof(jb));
        return true;
    }
    SmallJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.zero = zero; jb.nzero = zero ? nzero : 0;
    single_geometry(outer, n, inner, &jb);
    jb.nwg = nwg;
    SmallView& v = jb.v;
    v.U = U; v.part = part; v.n = n; v.r = r;
    v.sI = (int)inner; v.div = (int)inner; v.mulA = n * (int)inner; v.mulB = 1; v.cols_per_o = (int)inner;
    v.inv_div = 1.0f / (float)v.div;
    const int nbm = (n + 15) / 16, nbr = (r + 15) / 16;
    out->key = (xt == BF16 ? 1u : 0u) | ((unsigned)nbm << 4) | ((unsigned)nbr << 8);
    std::snprintf(out->label, sizeof(out->label), "k_subspace_small<%s, %d, %d>", tn, nbm, nbr);
    static_assert(sizeof(SmallJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

template <typename T>
static bool launch_small_t(const Batch<SmallJob>& b, dim3 grid, int nbm, int nbr, hipStream_t st) {
#define ASI_SS_CASE(M, R)                                                                      \
    if (nbm == M && nbr == R) {                                                                \
        hipLaunchKernelGGL((k_subspace_small<T, M, R>), grid, 256, 0, st, b);                  \
        return true;                                                                           \
    }
    ASI_SS_CASE(1, 1) ASI_SS_CASE(2, 1) ASI_SS_CASE(2, 2) ASI_SS_CASE(3, 1) ASI_SS_CASE(3, 2)
    ASI_SS_CASE(3, 3) ASI_SS_CASE(4, 1) ASI_SS_CASE(4, 2) ASI_SS_CASE(4, 3) ASI_SS_CASE(4, 4)
#undef ASI_SS_CASE
    return false;
}

hipError_t launch_small_items(const Item* const* items, int n, hipStream_t st) {
    const unsigned key = items[0]->key;
    dim3 grid;
    if (key & 4u) {
        Batch<ColsJob> b;
        if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
        switch (key & 3u) {
            case 0: hipLaunchKernelGGL((k_subspace_cols<float, false>), grid, SC_NT, SC_LDS, st, b); break;
            case 1: hipLaunchKernelGGL((k_subspace_cols<bf16_t, false>), grid, SC_NT, SC_LDS, st, b); break;
            case 2: hipLaunchKernelGGL((k_subspace_cols<float, true>), grid, SC_NT, SC_LDS, st, b); break;
            default: hipLaunchKernelGGL((k_subspace_cols<bf16_t, true>), grid, SC_NT, SC_LDS, st, b); break;
        }
        return hipGetLastError();
    }
    Batch<SmallJob> b;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const int nbm = (int)((key >> 4) & 7u), nbr = (int)((key >> 8) & 7u);
    const bool ok = (key & 1u) ? launch_small_t<bf16_t>(b, grid, nbm, nbr, st) : launch_small_t<float>(b, grid, nbm, nbr, st);
    return ok ? hipGetLastError() : hipErrorInvalidValue;
}

}  // namespace asi
