// m-mode product (Eq. 4) on fp32 MFMA:  Y[o,q,j] = sum_i X[o,i,j] M(i,q).
//
// Seen as a GEMM the unfolding's columns c = (o,j) are the long dimension, the mode index i
// is K and q is N.  A workgroup owns 64 columns and up to 64 outputs q; K is walked in
// chunks of 32 that are prefetched into registers while the previous chunk is multiplied
// (LDS double use, one barrier pair per chunk).  Wave w multiplies columns 16w..16w+15:
//   A operand (16 columns x 4 i)   = Xs[4ks + lane/16][16w + lane%16]
//   B operand (4 i x 16 q)         = Ms[4ks + lane/16][16nb + lane%16]
// The result tile is transposed through LDS so that stores run along the contiguous index.
// With KRON the matrix is the Kronecker product of two factors, M(i,q) = M1(i/n2, q/r2) *
// M2(i%n2, q%r2), which contracts two adjacent modes (H and W) in one pass.
//
// k_ttm_ksplit serves long fibres with few unfolding columns (the channel mode of a late conv
// layer): a workgroup owns 16 or 32 columns, its eight waves split the mode index between them, every operand goes from
// global memory straight into the MFMA registers, and the partial tiles are added through LDS.
//
// k_ttm_thin serves modes of at most 16 entries over very many columns on the vector ALU (further down).
//
// All kernels take the argument blocks of several layers side by side (Batch<TtmJob>).
#include "asi_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"
#include "asi_zplanes.h"

#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

typedef float v4f __attribute__((ext_vector_type(4)));

constexpr int TM_TC = 64, TM_TQ = 64;
// Row pitch of the LDS tiles in floats.  An operand read takes rows 4ks + lane / 16 at columns lane % 16 of
// a wave's block; a pitch of 16 banks more than a multiple of 64 puts the four rows on disjoint banks (a
// pitch of 68 puts them 4 banks apart: up to four lanes per bank).  Along the last mode the tile is stored
// transposed (lanes along the row index), where that pitch would send 16 lanes to one bank; an odd
// multiple of the bank width (17) spreads the rows of the store and keeps the reads nearly disjoint.
// Measured bank-conflict cycles per active LDS cycle: 0.08-0.24 (was 0.50) and 0.38-0.40 (was 0.54-0.60).
template <bool LASTMODE> constexpr int tm_ld() { return LASTMODE ? TM_TC + 17 : TM_TC + 16; }
constexpr int TM_LD_MAX = TM_TC + 17;
constexpr int TM_KCMAX = 64;

// KM: 0 = plain matrix, 1 = Kronecker product, 2 = Kronecker product with K chunks of 64 (long merged
// modes with few columns; otherwise chunks of 32, which overlap across workgroups), 3 = plain matrix with
// K chunks of 64 (a long last mode with at most one workgroup per CU: a chunk is a dependent round trip
// to memory, and nothing else on the CU hides it)
constexpr int TM_SMEM = 2 * TM_KCMAX * TM_LD_MAX;   // floats: Xs | Ms during the K loop, Ys (64 x TM_LD) afterwards

// one tile (workgroup lb of job jb); smem holds TM_SMEM floats
template <typename T, bool LASTMODE, int NBR, int KM>
__device__ __forceinline__ void ttm_tile(const TtmJob& jb, int lb, float* smem) {
    constexpr bool KRON = KM == 1 || KM == 2;
    constexpr int TM_KC = KM >= 2 ? 64 : 32;
    constexpr int TM_LR = TM_KC / 4;      // loads per thread and operand for one chunk
    constexpr int TM_LD = tm_ld<LASTMODE>();
    float (*Xs)[TM_LD] = reinterpret_cast<float (*)[TM_LD]>(smem);
    float (*Ms)[TM_LD] = reinterpret_cast<float (*)[TM_LD]>(smem + TM_KCMAX * TM_LD);
    float (*Ys)[TM_LD] = reinterpret_cast<float (*)[TM_LD]>(smem);
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const float* __restrict__ Mp = jb.Mp;
    float* __restrict__ Y = jb.Y;
    const long long outer = jb.outer, inner = jb.inner, ms_i = jb.ms_i, ms_q = jb.ms_q;
    const int n = jb.n, r = jb.r, beta = jb.beta;
    const KronSpec kr = jb.kr;
    const int bx = lb / jb.gy, by = lb - bx * jb.gy;      // output tiles of the same columns are neighbours (one L2)
    const long long ncols = outer * inner;
    const int tcols = jb.tile_cols;                  // columns of a tile in use (<= TM_TC)
    const long long c0 = (long long)bx * tcols;
    const int q0 = by * TM_TQ;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;

    // loader coordinates
    long long ld_base = -1;
    int l_c, l_i;
    if (!LASTMODE) {
        l_c = tid & 63; l_i = tid >> 6;              // rows l_i + 4t
        const long long c = c0 + l_c;
        if (c < ncols && l_c < tcols) {
            const long long o = c / inner, j = c - o * inner;
            ld_base = o * (long long)n * inner + j;
        }
    } else {
        l_i = tid & (TM_KC - 1); l_c = tid / TM_KC;   // columns l_c + (256 / TM_KC) t
    }
    const int m_q = tid & 63, m_i = tid >> 6;        // Ms loader: rows m_i + 4t
    // a matrix stored with the mode index contiguous (the transposed factor of step 5 of Eq. 14) is
    // loaded with the lanes along that index instead: row tid % KC, outputs tid / KC + (256 / KC) t
    const bool m_tr = !KRON && ms_i == 1 && ms_q != 1;
    const int t_i = tid & (TM_KC - 1), t_q = tid / TM_KC;

    // Kronecker indices by a rounded float quotient: exact for arguments below 2^14 (checked on the host)
    const float inv_n2 = 1.0f / (float)kr.n2, inv_r2 = 1.0f / (float)kr.r2;

    v4f acc[NBR];
#pragma unroll
    for (int nb = 0; nb < NBR; ++nb) acc[nb] = (v4f){0.f, 0.f, 0.f, 0.f};

    // The K loop, compiled once per matrix layout (MTR) so that the layout is no test inside it.
    auto kloop = [&](auto mtr_c) {
        constexpr bool MTR = decltype(mtr_c)::value;
        // Every load goes to an address that is always valid: a lane outside the tile reads the tile's
        // first column / first output instead, a row past n reads row n - 1.  What the loads return
        // stays untouched in registers until stash() masks and widens it, after the previous chunk's
        // MFMAs: the chunk's loads are one straight run of instructions, all in flight together, and
        // nothing waits for one of them before the multiply.
        T xr[TM_LR];
        float mr[TM_LR], m2[KRON ? TM_LR : 1];
        const bool x_in = LASTMODE ? true : ld_base >= 0;
        long long x_org;                              // element index of (this lane's column, row 0 / l_i)
        if (!LASTMODE) {
            const long long o = c0 / inner, j = c0 - o * inner;
            x_org = x_in ? ld_base : o * (long long)n * inner + j;
        } else {
            x_org = c0 * (long long)n;
        }
        const bool qm_in = q0 + m_q < r;                             // plain and Kronecker layouts
        const int qm = qm_in ? q0 + m_q : q0;
        const int qm1 = (int)(((float)qm + 0.5f) * inv_r2), qm2 = qm - qm1 * kr.r2;
        // PART: the chunk may reach past n (rows are clamped, empty row groups skipped: a uniform test);
        // otherwise it lies wholly below n and no test on the mode index remains
        auto fetch = [&](int k0, auto part_c) {
            constexpr bool PART = decltype(part_c)::value;
            auto row = [&](int i) { return (PART && i >= n) ? n - 1 : i; };
#pragma unroll
            for (int t = 0; t < TM_LR; ++t) {
                const bool live = !PART || k0 + 4 * t < n;
                if (!LASTMODE) {
                    if (live) xr[t] = X[x_org + (long long)row(k0 + l_i + 4 * t) * inner];
                    else xr[t] = T{};
                } else {
                    const int cl = l_c + (256 / TM_KC) * t;
                    const bool in = c0 + cl < ncols && cl < tcols;
                    xr[t] = X[x_org + row(k0 + l_i) + (in ? (long long)cl * n : 0LL)];
                }
                if (MTR) {
                    const int qt = q0 + t_q + (256 / TM_KC) * t;
                    mr[t] = Mp[(long long)row(k0 + t_i) + (long long)(qt < r ? qt : q0) * ms_q];
                } else if (!live) {
                    mr[t] = 0.f;
                    if (KRON) m2[t] = 0.f;
                } else if (!KRON) {
                    mr[t] = Mp[(long long)row(k0 + m_i + 4 * t) * ms_i + (long long)qm * ms_q];
                } else {
                    const int i = row(k0 + m_i + 4 * t);
                    const int i1 = (int)(((float)i + 0.5f) * inv_n2), i2 = i - i1 * kr.n2;
                    mr[t] = Mp[(long long)i1 * ms_i + (long long)qm1 * ms_q];
                    m2[t] = kr.M2[(long long)i2 * kr.ms_i + (long long)qm2 * kr.ms_q];
                }
            }
        };
        auto stash = [&](int k0) {
#pragma unroll
            for (int t = 0; t < TM_LR; ++t) {
                if (!LASTMODE) {
                    Xs[l_i + 4 * t][l_c] = (x_in && k0 + l_i + 4 * t < n) ? to_f32(xr[t]) : 0.f;
                } else {
                    const int cl = l_c + (256 / TM_KC) * t;
                    Xs[l_i][cl] = (c0 + cl < ncols && cl < tcols && k0 + l_i < n) ? to_f32(xr[t]) : 0.f;
                }
                if (MTR) {
                    const int ql = t_q + (256 / TM_KC) * t;
                    Ms[t_i][ql] = (q0 + ql < r && k0 + t_i < n) ? mr[t] : 0.f;
                } else {
                    const float v = KRON ? mr[t] * m2[t] : mr[t];
                    Ms[m_i + 4 * t][m_q] = (qm_in && k0 + m_i + 4 * t < n) ? v : 0.f;
                }
            }
        };
        // operands of two K steps at a time, read one group ahead of the MFMAs that use them
        constexpr int GS = 2, NG = TM_KC / 4 / GS;
        auto operands = [&](int g, float (&a)[GS], float (&b)[GS][NBR]) {
#pragma unroll
            for (int s = 0; s < GS; ++s) {
                a[s] = Xs[4 * (GS * g + s) + lg][16 * wave + ll];
#pragma unroll
                for (int nb = 0; nb < NBR; ++nb) b[s][nb] = Ms[4 * (GS * g + s) + lg][16 * nb + ll];
            }
        };
        auto multiply = [&](const float (&a)[GS], const float (&b)[GS][NBR]) {
#pragma unroll
            for (int s = 0; s < GS; ++s)
#pragma unroll
                for (int nb = 0; nb < NBR; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[s], b[s][nb], acc[nb], 0, 0, 0);
        };

        const std::true_type partial{};
        const std::false_type whole{};
        if (TM_KC <= n) fetch(0, whole); else fetch(0, partial);
        for (int k0 = 0; k0 < n; k0 += TM_KC) {
            __syncthreads();                 // previous chunk fully consumed
            stash(k0);
            __syncthreads();
            const int nx = k0 + TM_KC;
            if (nx + TM_KC <= n) fetch(nx, whole);
            else if (nx < n) fetch(nx, partial);
            if (nx <= n) {
                float a0[GS], b0[GS][NBR], a1[GS], b1[GS][NBR];
                // (scheduling fences: without them the compiler moves every read back next to its MFMA
                // and waits for it there)
                operands(0, a0, b0);
#pragma unroll
                for (int g = 0; g < NG; g += 2) {
                    operands(g + 1, a1, b1);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(a0, b0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (g + 2 < NG) operands(g + 2, a0, b0);
                    __builtin_amdgcn_sched_barrier(0);
                    multiply(a1, b1);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int ks = 0; ks < TM_KC / 4; ++ks) {
                    if (k0 + 4 * ks < n) {
                        const float a = Xs[4 * ks + lg][16 * wave + ll];
#pragma unroll
                        for (int nb = 0; nb < NBR; ++nb)
                            acc[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, Ms[4 * ks + lg][16 * nb + ll], acc[nb], 0, 0, 0);
                    }
                }
            }
        }
    };
    if (m_tr) kloop(std::true_type{}); else kloop(std::false_type{});
    __syncthreads();
    // result layout: lane holds column 16w + 4*lg + v, output 16nb + ll
#pragma unroll
    for (int nb = 0; nb < NBR; ++nb)
#pragma unroll
        for (int v = 0; v < 4; ++v) Ys[16 * nb + ll][16 * wave + 4 * lg + v] = acc[nb][v];
    __syncthreads();
    const int rq = (r - q0 < TM_TQ) ? r - q0 : TM_TQ;
    if (!LASTMODE && inner < TM_TC) {
        // short inner extent: a tile holds whole outer indices, and for one outer index the (q, j)
        // pairs of this workgroup are one contiguous run of Y
        const int k_o = tcols / (int)inner;
        const long long o0 = (long long)bx * k_o;
        const int nvo = (int)((outer - o0 < k_o) ? outer - o0 : k_o);
        const int run = rq * (int)inner, total = nvo * run;          // total <= 4096: float quotients are exact
        const float inv_run = 1.0f / (float)run, inv_in = 1.0f / (float)inner;
        for (int e = tid; e < total; e += 256) {
            const int ol = (int)(((float)e + 0.5f) * inv_run), rem = e - ol * run;
            const int ql = (int)(((float)rem + 0.5f) * inv_in), j = rem - ql * (int)inner;
            const long long idx = ((o0 + ol) * r + q0) * inner + rem;
            const float v = Ys[ql][ol * (int)inner + j];
            Y[idx] = beta ? Y[idx] + v : v;
        }
    } else if (!LASTMODE) {
        const int cl = tid & 63;
        const long long c = c0 + cl;
        if (c < ncols && cl < tcols) {
            const long long o = c / inner, j = c - o * inner;
            for (int ql = tid >> 6; ql < rq; ql += 4) {
                const long long idx = (o * r + q0 + ql) * inner + j;
                Y[idx] = beta ? Y[idx] + Ys[ql][cl] : Ys[ql][cl];
            }
        }
    } else {
        for (int e = tid; e < TM_TC * rq; e += 256) {
            const int cl = e / rq, ql = e - cl * rq;
            const long long c = c0 + cl;
            if (c < ncols && cl < tcols) {
                const long long idx = c * r + q0 + ql;
                Y[idx] = beta ? Y[idx] + Ys[ql][cl] : Ys[ql][cl];
            }
        }
    }
}

template <typename T, bool LASTMODE, int NBR, int KM>
__global__ __launch_bounds__(256) void k_ttm_mfma(Batch<TtmJob> bt) {
    __shared__ float smem[TM_SMEM];
    int lb;
    const TtmJob& jb = bt.job[locate_xcd(bt, &lb)];
    ttm_tile<T, LASTMODE, NBR, KM>(jb, lb, smem);
}

// Two independent products in one launch: a plain product along a leading mode (G1 = grad_out x_1 U1^T
// of Eq. 14) and, in extra workgroups, Z = S x_3 U3 x_4 U4 plane by plane or, KRON, as one merged product (a row or a column longer
// than 64, a rank above 32: signals of 1 x 200, apart 3 us longer).
template <bool KRON>
struct TtmDuoJob {
    TtmJob a;        // dtype T, not the last mode, plain matrix, NBR column blocks
    std::conditional_t<KRON, TtmJob, ZPlanesJob> z;      // (KRON: fp32, trailing modes merged by a Kronecker product, K chunks of 32)
    int a_blocks;
};
template <typename T, int NBR, bool KRON>
__global__ __launch_bounds__(256) void k_ttm_duo(Batch<TtmDuoJob<KRON>> bt) {
    __shared__ float smem[TM_SMEM];
    int lb;
    const TtmDuoJob<KRON>& jb = bt.job[locate(bt, &lb)];
    if (lb < jb.a_blocks) ttm_tile<T, false, NBR, 0>(jb.a, xcd_order(lb, jb.a_blocks), smem);
    else if constexpr (KRON) ttm_tile<float, true, 4, 1>(jb.z, lb - jb.a_blocks, smem);
    else z_planes_block<0, false>(jb.z, lb - jb.a_blocks);
}

// ---- long fibres, few columns ------------------------------------------------------------------
// A workgroup owns 16 CB columns (CB: one or two); its NW waves (eight or four) deal the K steps (four mode indices each) of the whole mode among
// themselves, and every operand goes from memory straight into the registers of the lanes that multiply it:
//   A operand (16 columns x 4 i)  = X at row 4 s + lane / 16 of column 16 cb + lane % 16
//   B operand (4 i x 16 outputs)  = M at row 4 s + lane / 16; lane ll of a row holds the NBR CONSECUTIVE outputs NBR ll + nb, one
//                                   load of 4 NBR bytes for NBR blocks of interleaved outputs.  CONTIG = false, the matrix stored the other
//                                   way round: outputs 16 nb + ll, so that the 16 rows of a load follow each other in memory, and no load
//                                   for steps past the wave's last (the loads are the bound: 130 x 400 over 2304 columns 33.4 -> 16.7 us,
//                                   the order of outputs alone 22.4 -> 16.7)
// What bounds it is the number of loads between a workgroup's start and its end, not the products: R steps are requested while
// the R before them are multiplied.  With four waves, 16 columns, a dword per operand and no step requested ahead a 960-long
// mode took 180 + 60 loads a wave in four dependent rounds, here 30 x (1 + CB): 960 x 40 over 6272 columns (24 MB) 17.9 -> 13.6 us,
// 512 x 48 over 3 x 3136 (19 MB) 19.7 -> 13.5, 256 x 32 over 12544 (13 MB) 10.0 -> 6.7.  At 960 the products are 4.8 us of it (196
// workgroups, 180 of them a SIMD and wave).  M is read through a buffer
// descriptor: what lies beyond its last element arrives as zero (a row beyond the mode, or the next row's entries in outputs that
// are dropped anyway), so neither needs a test in the loop; a last step that is not whole is masked by itself.
template <int N> struct LoadB;
template <> struct LoadB<1> { typedef unsigned type; };
template <> struct LoadB<2> { typedef unsigned type __attribute__((ext_vector_type(2))); };
template <> struct LoadB<3> { typedef unsigned type __attribute__((ext_vector_type(3))); };
template <> struct LoadB<4> { typedef unsigned type __attribute__((ext_vector_type(4))); };

template <typename T, int NBR, int CB, bool CONTIG, int NW>
__global__ __launch_bounds__(64 * NW, 4) void k_ttm_ksplit(Batch<TtmJob> bt) {
    // steps in flight beside those being multiplied (128 registers); a matrix stored the other way round is bound by the loads themselves
    constexpr int R = !CONTIG ? 2 : NBR + CB <= 4 ? 8 : 36 / (NBR + CB);
    constexpr int LD = 16 * CB + 4;                  // pitch of a partial tile's row: 16-byte pieces stay aligned
    extern __shared__ __align__(16) float ks_red[];  // [NW][16 NBR][LD]
    int lb;
    const TtmJob& jb = bt.job[locate_xcd(bt, &lb)];
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    float* __restrict__ Y = jb.Y;
    const long long outer = jb.outer, inner = jb.inner;
    const int n = jb.n, r = jb.r, beta = jb.beta;
    const unsigned ms_i = (unsigned)jb.ms_i, ms_q = (unsigned)jb.ms_q;        // the matrix is below 2 GB (host check)
    const int bx = lb / jb.gy, by = lb - bx * jb.gy;      // output tiles of the same columns are neighbours (one L2)
    const long long ncols = outer * inner;
    const long long c0 = (long long)bx * (16 * CB);
    const int q0 = by * (NBR * 16);
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;
    // this lane's columns, as 32-bit offsets from the workgroup's first slab (host check)
    const long long o0 = c0 / inner;
    const T* __restrict__ Xw = X + o0 * (long long)n * inner;
    unsigned xoff[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) {
        const long long c = c0 + 16 * cb + ll, cc = c < ncols ? c : c0;       // past the end: the first column, dropped at the store
        const long long o = cc / inner, j = cc - o * inner;
        xoff[cb] = (unsigned)((o - o0) * (long long)n * inner + j);
    }
    const unsigned row = (unsigned)inner;
    const unsigned qoff = (unsigned)(q0 + (CONTIG ? NBR * ll : ll)) * ms_q;
    const int steps = (n + 3) >> 2;
    const int mine = wave < steps ? (steps - 1 - wave) / NW + 1 : 0;       // steps wave, wave + 8, ..
    const bool ragged = (n & 3) != 0;
#if defined(__HIP_DEVICE_COMPILE__)
    const auto mrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(jb.Mp), 0, (int)(4u * ((unsigned)(n - 1) * ms_i + (unsigned)(r - 1) * ms_q + 1u)), 0x00027000);
#endif
    typedef typename LoadB<NBR>::type MV;
    struct Stage { T x[R][CB]; MV m[R]; };
    auto fetch = [&](int t0, Stage& g) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < R; ++u) {
            if (!CONTIG && t0 + u >= mine) continue;
            const int t = t0 + u < mine ? t0 + u : mine - 1;                  // uniform; a repeated step is not multiplied
            const int i0 = 4 * (wave + NW * t), i = i0 + lg;
            const unsigned xr = (unsigned)(i < n ? i : n - 1) * row;
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) g.x[u][cb] = Xw[xoff[cb] + xr];
#if defined(__HIP_DEVICE_COMPILE__)
            const int mo = (int)(4u * ((unsigned)i * ms_i + qoff));
            if (CONTIG) {
                if constexpr (NBR == 1) g.m[u] = __builtin_amdgcn_raw_buffer_load_b32(mrsrc, mo, 0, 0);
                if constexpr (NBR == 2) g.m[u] = __builtin_amdgcn_raw_buffer_load_b64(mrsrc, mo, 0, 0);
                if constexpr (NBR == 3) g.m[u] = __builtin_amdgcn_raw_buffer_load_b96(mrsrc, mo, 0, 0);
                if constexpr (NBR == 4) g.m[u] = __builtin_amdgcn_raw_buffer_load_b128(mrsrc, mo, 0, 0);
            } else {
                unsigned e[NBR];
#pragma unroll
                for (int nb = 0; nb < NBR; ++nb) e[nb] = __builtin_amdgcn_raw_buffer_load_b32(mrsrc, mo + (int)(64u * nb * ms_q), 0, 0);
                __builtin_memcpy(&g.m[u], e, sizeof(e));
            }
#endif
        }
    };
    v4f acc[CB][NBR];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int nb = 0; nb < NBR; ++nb) acc[cb][nb] = (v4f){0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int t0, Stage& g) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < R; ++u)
            if (t0 + u < mine) {                     // uniform
                const int s = wave + NW * (t0 + u);
                float x[CB], m[NBR];
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) x[cb] = to_f32(g.x[u][cb]);
                __builtin_memcpy(m, &g.m[u], sizeof(m));
                if (ragged && s == steps - 1) {      // uniform
                    const bool in = 4 * s + lg < n;
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) x[cb] = in ? x[cb] : 0.f;
#pragma unroll
                    for (int nb = 0; nb < NBR; ++nb) m[nb] = in ? m[nb] : 0.f;
                }
#pragma unroll
                for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                    for (int nb = 0; nb < NBR; ++nb)
                        acc[cb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[cb], m[nb], acc[cb][nb], 0, 0, 0);
            }
    };
    if (mine > 0) {
        Stage a, b;
        fetch(0, a);
        for (int t = 0; t < mine; t += 2 * R) {
            if (t + R < mine) fetch(t + R, b);
            multiply(t, a);
            if (t + R < mine) {
                if (t + 2 * R < mine) fetch(t + 2 * R, a);
                multiply(t + R, b);
            }
        }
    }
    // lane holds columns 16 cb + 4 lg .. + 3, output NBR ll + nb
#pragma unroll
    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
        for (int nb = 0; nb < NBR; ++nb)
            *reinterpret_cast<v4f*>(ks_red + (wave * 16 * NBR + (CONTIG ? NBR * ll + nb : 16 * nb + ll)) * LD + 16 * cb + 4 * lg) = acc[cb][nb];
    __syncthreads();
    constexpr int W = 16 * CB;
    const int cl = tid % W;
    const long long cc = c0 + cl;
    if (cc < ncols) {
        const long long o = cc / inner, j = cc - o * inner;
        for (int ql = tid / W; ql < NBR * 16; ql += 64 * NW / W) {
            const int q = q0 + ql;
            if (q < r) {
                float p[8] = {};
#pragma unroll
                for (int w = 0; w < NW; ++w) p[w] = ks_red[(w * 16 * NBR + ql) * LD + cl];
                float v = (p[0] + p[1]) + (p[2] + p[3]);
                if (NW == 8) v += (p[4] + p[5]) + (p[6] + p[7]);
                const long long idx = (o * r + q) * inner + j;
                Y[idx] = beta ? Y[idx] + v : v;
            }
        }
    }
}

// ---- very short modes on the vector ALU ---------------------------------------------------------
// A mode of at most 16 entries with at most 16 outputs (the batch mode of a high-resolution layer:
// 8 x 8 over a million columns) gives the MFMA tiles of k_ttm_mfma nothing to do — a 64-column tile is
// 2 KB of data, and the launch is bound by the number of workgroups.  Here a thread owns TH_CPT
// columns: it loads their n values (lanes along the contiguous index), multiplies by the matrix held
// in LDS (read as whole rows, the same address in every lane) and stores r values per column.
constexpr int TH_CPT = 2, TH_COLS = 256 * TH_CPT;
template <typename T, int NMAX>
__global__ __launch_bounds__(256) void k_ttm_thin(Batch<TtmJob> bt) {
    __shared__ __align__(16) float Ms[16][16];
    int lb;
    const TtmJob& jb = bt.job[locate(bt, &lb)];
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    float* __restrict__ Y = jb.Y;
    const long long outer = jb.outer, inner = jb.inner, ncols = outer * inner;
    const int n = jb.n, r = jb.r, beta = jb.beta, tid = threadIdx.x;
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;
    {
        const int i = tid >> 4, q = tid & 15;
        Ms[i][q] = ldg_f32(jb.Mp, (long long)i * jb.ms_i + (long long)q * jb.ms_q, i < n && q < r);
    }
    // (o, j) of the workgroup's first column by one division (uniform), of a thread's columns by additions
    const long long cw = (long long)lb * TH_COLS;
    const long long ow = cw / inner, jw = cw - ow * inner;
    long long xb[TH_CPT], yb[TH_CPT];
    bool ok[TH_CPT];
    T xv[TH_CPT][NMAX];
#pragma unroll
    for (int t = 0; t < TH_CPT; ++t) {
        long long o = ow, j = jw + t * 256 + tid;
        while (j >= inner) { j -= inner; ++o; }
        ok[t] = cw + t * 256 + tid < ncols;
        xb[t] = ok[t] ? o * (long long)n * inner + j : 0;          // past the end: column 0, dropped at the store
        yb[t] = ok[t] ? o * (long long)r * inner + j : 0;
#pragma unroll
        for (int i = 0; i < NMAX; ++i) xv[t][i] = X[xb[t] + (long long)(i < n ? i : n - 1) * inner];
    }
    __syncthreads();
    float acc[TH_CPT][16];
#pragma unroll
    for (int t = 0; t < TH_CPT; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[t][q] = 0.f;
#pragma unroll
    for (int i = 0; i < NMAX; ++i) {
        float m[16];
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
            const v4f row = *reinterpret_cast<const v4f*>(&Ms[i][4 * q4]);      // rows i >= n are zero
            m[4 * q4] = row[0]; m[4 * q4 + 1] = row[1]; m[4 * q4 + 2] = row[2]; m[4 * q4 + 3] = row[3];
        }
#pragma unroll
        for (int t = 0; t < TH_CPT; ++t) {
            const float x = i < n ? to_f32(xv[t][i]) : 0.f;
#pragma unroll
            for (int q = 0; q < 16; ++q) acc[t][q] = fmaf(x, m[q], acc[t][q]);
        }
    }
#pragma unroll
    for (int t = 0; t < TH_CPT; ++t)
#pragma unroll
        for (int q = 0; q < 16; ++q)
            if (ok[t] && q < r) {
                const long long idx = yb[t] + (long long)q * inner;
                Y[idx] = beta ? Y[idx] + acc[t][q] : acc[t][q];
            }
}

// ---- a short last mode expanded to many outputs ------------------------------------------------
// Y[c, q] (+)= sum_k X[c, k] M(k, q) with at most 32 terms and 256 or more outputs per column: the last
// step of the linear weight gradient (dW = T U_3^T: rank 20, thousands of features).  The output is the
// only large tensor, so the kernel is built around its stores: a workgroup owns 256 outputs and walks `tile_cols` columns in
// passes of 32; M's tile is staged once, the next pass's X tile is requested before the products of this one.  Products run
// on the fp32 MFMA, rows = outputs (a lane then holds four consecutive ones), a wave 64 outputs x 32 columns; the tile goes
// through LDS so that a store instruction writes 1 KB of one output row.  On the vector ALU (a thread per four outputs of
// eight columns) every multiply-add needed its share of nine LDS reads per term: 22.8 -> 19.5 us for 5632 x 2048 outputs of
// rank 20 (46 MB written).
constexpr int EX_C = 32, EX_Q = 256, EX_K = 32, EX_YP = EX_Q + 4;
__global__ __launch_bounds__(256) void k_ttm_expand(Batch<TtmJob> bt) {
    constexpr int MP = EX_Q + 16;                    // pitch 16 mod 32: the two row groups of a half wave lie on other banks
    __shared__ __align__(16) float ex_tile[EX_K * MP];       // M's tile, then the result tile of a pass
    __shared__ float Xs[EX_C][EX_K + 1];
    static_assert(EX_C * EX_YP <= EX_K * MP, "the result tile takes the place of M's");
    float (*Ms)[MP] = reinterpret_cast<float (*)[MP]>(ex_tile);
    float (*Ys)[EX_YP] = reinterpret_cast<float (*)[EX_YP]>(ex_tile);
    int lb;
    const TtmJob& jb = bt.job[locate(bt, &lb)];
    const float* __restrict__ X = static_cast<const float*>(jb.X);
    const float* __restrict__ Mp = jb.Mp;
    float* __restrict__ Y = jb.Y;
    const long long ncols = jb.outer, ms_i = jb.ms_i, ms_q = jb.ms_q;
    const int n = jb.n, r = jb.r, beta = jb.beta, n4 = (n + 3) & ~3;
    const int bx = lb / jb.gy, by = lb - bx * jb.gy;
    const long long c0 = (long long)bx * jb.tile_cols;
    const int q0 = by * EX_Q;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;
    // tiles: consecutive threads along the index that is contiguous in memory; every load of the workgroup is
    // issued before the first is stored (clamped addresses, masks at the store: nothing waits in between)
    const bool k_fast = ms_i == 1;
    const float inv_n = 1.0f / (float)n;             // e < 2^13: the rounded float quotients are exact
    float mt[EX_K], xt[EX_C * EX_K / 256];
    auto x_load = [&](long long cb) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < EX_C * EX_K / 256; ++u) {
            const int e = tid + 256 * u;
            const int c = (int)(((float)e + 0.5f) * inv_n);
            xt[u] = X[e < EX_C * n && cb + c < ncols ? cb * n + e : 0LL];
        }
    };
#pragma unroll
    for (int u = 0; u < EX_K; ++u) {
        const int e = tid + 256 * u;
        const int eq = (int)(((float)e + 0.5f) * inv_n);
        const int k = k_fast ? e - eq * n : u, q = k_fast ? eq : tid;       // (e / 256 = u, e % 256 = tid)
        const bool ok = e < EX_Q * n && q0 + q < r;
        mt[u] = Mp[ok ? (long long)k * ms_i + (long long)(q0 + q) * ms_q : 0LL];
    }
    x_load(c0);
    for (int e = tid; e < (n4 - n) * EX_Q; e += 256) Ms[n + (e >> 8)][e & 255] = 0.f;        // terms up to a multiple of four
    for (int e = tid; e < (n4 - n) * EX_C; e += 256) Xs[e & 31][n + (e >> 5)] = 0.f;
#pragma unroll
    for (int u = 0; u < EX_K; ++u) {
        const int e = tid + 256 * u;
        const int eq = (int)(((float)e + 0.5f) * inv_n);
        const int k = k_fast ? e - eq * n : u, q = k_fast ? eq : tid;
        if (e < EX_Q * n) Ms[k][q] = (q0 + q < r) ? mt[u] : 0.f;
    }
    __syncthreads();
    float a[EX_K / 4][4];                            // the wave's A operands: 64 outputs, all terms
#pragma unroll
    for (int ks = 0; ks < EX_K / 4; ++ks)
#pragma unroll
        for (int t = 0; t < 4; ++t) a[ks][t] = 4 * ks < n4 ? Ms[4 * ks + lg][64 * wave + 16 * t + ll] : 0.f;
    const int np = jb.tile_cols / EX_C;
    for (int p = 0; p < np; ++p) {
        const long long cb = c0 + p * EX_C;
        if (cb >= ncols) break;
#pragma unroll
        for (int u = 0; u < EX_C * EX_K / 256; ++u) {
            const int e = tid + 256 * u;
            const int c = (int)(((float)e + 0.5f) * inv_n), k = e - c * n;
            if (e < EX_C * n) Xs[c][k] = (cb + c < ncols) ? xt[u] : 0.f;
        }
        __syncthreads();                             // (also: M's tile and the last pass's result tile have been read)
        if (p + 1 < np) x_load(cb + EX_C);
        v4f acc[4][2];
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) acc[t][h] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < EX_K / 4; ++ks)
            if (4 * ks < n4) {
                float b[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) b[h] = Xs[16 * h + ll][4 * ks + lg];
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int h = 0; h < 2; ++h) acc[t][h] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[ks][t], b[h], acc[t][h], 0, 0, 0);
            }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int h = 0; h < 2; ++h) *reinterpret_cast<v4f*>(&Ys[16 * h + ll][64 * wave + 16 * t + 4 * lg]) = acc[t][h];
        __syncthreads();
        const int q = q0 + 4 * lane;
        if (q < r) {                                 // r is a multiple of four (host check): a piece is whole
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const long long c = cb + 8 * wave + j;
                if (c < ncols) {
                    v4f* yp = reinterpret_cast<v4f*>(Y + c * r + q);
                    v4f out = *reinterpret_cast<const v4f*>(&Ys[8 * wave + j][4 * lane]);
                    if (beta) out += *yp;
                    *yp = out;
                }
            }
        }
    }
}
static bool ttm_expand_supported(DType xt, long long inner, int n, int r, const float* Y) {
    return xt == F32 && inner == 1 && n <= EX_K && r >= EX_Q && r % 4 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0;
}

// ---- host side -----------------------------------------------------------------------------------
// key bits: [0] bf16 input, [1] LASTMODE, [2] KRON, [3] split kernel, [4..6] NBR-1,
// [14] K chunks of 64 (tiled kernel along the last mode), [15] the vector-ALU kernel for very short modes,
// [16] split kernel: two column blocks per workgroup, [17] four waves, [18] rows of the matrix contiguous.
// Bits 4..6 only bound sizes.
static unsigned ttm_key(bool bf16, bool last, bool kron, bool ksplit, int nbr, bool kc64) {
    return (bf16 ? 1u : 0u) | (last ? 2u : 0u) | (kron ? 4u : 0u) | (ksplit ? 8u : 0u) | ((unsigned)(nbr - 1) << 4) | (kc64 ? 0x4000u : 0u);
}

// The tiled kernel walks the mode index in n/32 dependent steps with ncols/64 workgroups; when that
// leaves most of the chip idle the split kernel is the faster one.
static bool prefer_ksplit(long long ncols, int n, long long inner) {
    return inner > 1 && n > 64 && (ncols + TM_TC - 1) / TM_TC < 512;
}

// its offsets have 32 bits, relative to the first slab of a workgroup's columns and to the matrix
static bool ksplit_reaches(long long outer, int n, long long inner, long long ms_i, long long ms_q, int r) {
    const long long slabs = 64 / inner + 2 < outer ? 64 / inner + 2 : outer;
    return ms_i > 0 && ms_q > 0 && slabs * n * inner < (1LL << 30) && (n + 3) * ms_i + (r + 63) * ms_q < (1LL << 29);
}
// Waves: eight for long modes, whose chain of steps is what a launch waits for; four up to 160 entries, of which eight waves would get two to
// five steps each and pay the sum of eight partial tiles for them (one layer of 77 x 3 over 11280 columns 7.6 -> 6.4 us, eight 28.4 -> 13.9 with the two
// column blocks below, G1 of 100 x 20 over 9800 columns eight times 32.6 -> 16.3; 200 entries 17.4 -> 14.9 in eight layers but 6.8 -> 8.3 in one),
// and for a matrix stored the other way round, whose loads of a row per lane are the bound (190 entries 25.5 -> 18.7).
static int ksplit_waves(int n, bool contig) { return n <= 160 || !contig ? 4 : 8; }
// Column blocks per workgroup.  Eight waves: the fewest column blocks that a CU multiplies one after the other, two a workgroup on a tie (they
// share the loads of the matrix).  One | two: 512 x 48 over 3 x 3136 columns (588 | 294 workgroups) 13.5 | 15.0 us, 960 x 40 over 6272 (392 |
// 196) 14.8 | 13.6, 256 x 32 over 12544 (784 | 392) 8.9 | 6.7; four: 9.2 there.  Four waves, of which a CU holds several workgroups: two as well where
// that leaves every CU one (130 x 400 over 9000 columns 46.5 -> 33.5 us, 77 x 3 over 3 x 11280 9.4 -> 8.7; with 256 it changes nothing).
static int ksplit_cb(long long ncols, int nw) {
    if (nw == 4 && (ncols + 15) / 16 >= 512) return 2;
    const long long one = ((ncols + 15) / 16 + 255) / 256, two = ((ncols + 31) / 32 + 255) / 256 * 2;
    return one < two ? 1 : 2;
}

static bool fill_ttm(DType xt, const void* X, long long outer, int n, long long inner, const float* Mp, long long ms_i,
                     long long ms_q, int r, float* Y, int beta, const KronSpec& kr, Item* out) {
    const long long ncols = outer * inner;
    if (ncols <= 0 || n <= 0 || r <= 0 || !X || !Mp || !Y) return false;
    const bool last = (inner == 1), kron = kr.M2 != nullptr;
    TtmJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.outer = outer; jb.inner = inner; jb.Mp = Mp; jb.ms_i = ms_i; jb.ms_q = ms_q; jb.Y = Y;
    jb.kr = kr; jb.n = n; jb.r = r; jb.beta = beta;
    const char* tn = xt == F32 ? "float" : "asi::bf16_t";
    *out = Item();
    if (!kron && ttm_expand_supported(xt, inner, n, r, Y)) {
        // two passes per workgroup once that still leaves two workgroups per CU: M's tile is then staged half as often
        const long long tiles = (ncols + EX_C - 1) / EX_C * ((r + EX_Q - 1) / EX_Q);
        jb.tile_cols = tiles >= 1024 ? 2 * EX_C : EX_C;
        const long long gx = (ncols + jb.tile_cols - 1) / jb.tile_cols;
        jb.gx = (int)gx; jb.gy = (r + EX_Q - 1) / EX_Q;
        if (gx * jb.gy > 0x3fffffffLL) return false;
        out->kind = IT_TTM_EXPAND; out->key = 0;
        std::snprintf(out->label, sizeof(out->label), "k_ttm_expand");
    } else if (!kron && !last && n <= 16 && r <= 16 && ncols >= (1LL << 18)) {
        const long long gx = (ncols + TH_COLS - 1) / TH_COLS;
        if (gx > 0x3fffffffLL) return false;
        jb.gx = (int)gx; jb.gy = 1;
        out->kind = IT_TTM; out->key = ttm_key(xt == BF16, false, false, false, 1, false) | 0x8000u;
        std::snprintf(out->label, sizeof(out->label), "k_ttm_thin<%s, %d>", tn, n <= 8 ? 8 : 16);
    } else if (!kron && prefer_ksplit(ncols, n, inner) && ksplit_reaches(outer, n, inner, ms_i, ms_q, r)) {
        const bool contig = ms_q == 1;
        const int nw = ksplit_waves(n, contig), cb = ksplit_cb(ncols, nw);
        const int nbr = r >= 64 ? 4 : (r + 15) / 16;
        const long long gx = (ncols + 16 * cb - 1) / (16 * cb);
        jb.gx = (int)gx; jb.gy = (r + nbr * 16 - 1) / (nbr * 16);
        if (gx * jb.gy > 0x3fffffffLL) return false;
        out->kind = IT_KSPLIT; out->key = ttm_key(xt == BF16, false, false, true, nbr, false) | ((unsigned)(cb - 1) << 16) | (nw == 4 ? 0x20000u : 0u) | (contig ? 0x40000u : 0u);
        std::snprintf(out->label, sizeof(out->label), "k_ttm_ksplit<%s, %d, %d, %s, %d>", tn, nbr, cb, contig ? "true" : "false", nw);
    } else {
        // short inner extents: tiles of whole outer indices (stores then run contiguously)
        jb.tile_cols = (!last && inner < TM_TC) ? (int)(TM_TC / inner * inner) : TM_TC;
        const long long gx = (!last && inner < TM_TC) ? (outer + TM_TC / inner - 1) / (TM_TC / inner)
                                                      : (ncols + TM_TC - 1) / TM_TC;
        const int rr = r < TM_TQ ? r : TM_TQ;
        const int nbr = (rr + 15) / 16;
        jb.gx = (int)gx; jb.gy = (r + TM_TQ - 1) / TM_TQ;
        if (gx * jb.gy > 0x3fffffffLL) return false;
        const bool kc64 = kron ? n > 64 : (last && n >= 256 && gx * jb.gy <= 256);   // (at most one workgroup per CU)
        out->kind = IT_TTM; out->key = ttm_key(xt == BF16, last, kron, false, nbr, kc64);
        std::snprintf(out->label, sizeof(out->label), "k_ttm_mfma<%s, %s, %d, %d>", tn, last ? "true" : "false", nbr,
                      kron ? (kc64 ? 2 : 1) : (kc64 ? 3 : 0));
    }
    out->nblocks = jb.gx * jb.gy;
    static_assert(sizeof(TtmJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

bool make_ttm(DType xt, const void* X, long long outer, int n, long long inner, const float* Mp, long long ms_i,
              long long ms_q, int r, float* Y, int beta, Item* out, bool stream_ok) {
    const KronSpec none = {nullptr, 0, 0, 1, 1};
    const long long ncols = outer * inner;
    const bool thin = n <= 16 && r <= 16 && ncols >= (1LL << 18);
    // the streaming kernel pays once the tensor is large enough to keep the chip busy with its loads
    // (the split kernel's 16-column workgroups spread few columns further: it keeps the products below 256 spans)
    if (stream_ok && inner > 1 && !thin && ncols * n >= kStreamMinElems && (ncols >= 256 * 64 || !prefer_ksplit(ncols, n, inner)) &&
        ttm_stream_supported(xt, X, outer, n, inner, Mp, ms_i, ms_q, r, Y))
        return make_ttm_stream(xt, X, outer, n, inner, Mp, ms_i, ms_q, r, Y, beta, out);
    return fill_ttm(xt, X, outer, n, inner, Mp, ms_i, ms_q, r, Y, beta, none, out);
}

bool make_ttm_kron(DType xt, const void* X, long long cols, int n1, int n2, const float* M1, long long ms1_i,
                   long long ms1_q, int r1, const float* M2, long long ms2_i, long long ms2_q, int r2, float* Y,
                   int beta, Item* out) {
    if (cols <= 0 || n1 <= 0 || n2 <= 0 || r1 <= 0 || r2 <= 0 || !M1 || !M2) return false;
    const KronSpec kr = {M2, ms2_i, ms2_q, n2, r2};
    return fill_ttm(xt, X, cols, n1 * n2, 1, M1, ms1_i, ms1_q, r1 * r2, Y, beta, kr, out);
}

template <typename T, bool LAST, int KM>
static void launch_tiled(int nbr, const Batch<TtmJob>& b, dim3 grid, hipStream_t st) {
    switch (nbr) {
        case 1: hipLaunchKernelGGL((k_ttm_mfma<T, LAST, 1, KM>), grid, 256, 0, st, b); break;
        case 2: hipLaunchKernelGGL((k_ttm_mfma<T, LAST, 2, KM>), grid, 256, 0, st, b); break;
        case 3: hipLaunchKernelGGL((k_ttm_mfma<T, LAST, 3, KM>), grid, 256, 0, st, b); break;
        default: hipLaunchKernelGGL((k_ttm_mfma<T, LAST, 4, KM>), grid, 256, 0, st, b); break;
    }
}
template <typename T, int NBR, int CB, bool CONTIG, int NW>
static hipError_t launch_split_one(const Batch<TtmJob>& b, dim3 grid, hipStream_t st) {
    constexpr size_t lds = sizeof(float) * NW * 16 * NBR * (16 * CB + 4);
    if (lds > 64 * 1024) {
        static LdsAllowed allowed;
        const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_ttm_ksplit<T, NBR, CB, CONTIG, NW>), lds, allowed);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_ttm_ksplit<T, NBR, CB, CONTIG, NW>), grid, 64 * NW, lds, st, b);
    return hipGetLastError();
}
template <typename T, int NBR, int CB>
static hipError_t launch_split_cb(int nw, bool contig, const Batch<TtmJob>& b, dim3 grid, hipStream_t st) {
    if (!contig) return nw == 4 ? launch_split_one<T, NBR, CB, false, 4>(b, grid, st) : hipErrorInvalidValue;
    return nw == 8 ? launch_split_one<T, NBR, CB, true, 8>(b, grid, st) : launch_split_one<T, NBR, CB, true, 4>(b, grid, st);
}
template <typename T, int NBR>
static hipError_t launch_split(int cb, int nw, bool contig, const Batch<TtmJob>& b, dim3 grid, hipStream_t st) {
    if (cb == 2) return launch_split_cb<T, NBR, 2>(nw, contig, b, grid, st);
    if (cb == 1) return launch_split_cb<T, NBR, 1>(nw, contig, b, grid, st);
    return hipErrorInvalidValue;
}

// a: a tiled plain product that is not along the last mode, with planes (make_z_planes) or a Kronecker product with short K as z, or a
// streaming one with planes.  Fails (and leaves *out alone) if they do not have these forms; the caller then launches them apart.
// key: [0] bf16, [1] KRON, [4..6] NBR-1
template <bool KRON>
static bool put_ttm_duo(const Item& a, const Item& z, Item* out) {
    typedef TtmDuoJob<KRON> J;
    J jb;
    std::memset(&jb, 0, sizeof(jb));
    std::memcpy(&jb.a, a.arg, sizeof(jb.a));
    std::memcpy(&jb.z, z.arg, sizeof(jb.z));
    jb.a_blocks = a.nblocks;
    if ((long long)a.nblocks + z.nblocks > 0x3fffffffLL) return false;
    const int nbr = (int)((a.key >> 4) & 7u) + 1;
    Item it;
    it.kind = IT_TTM_DUO;
    it.key = (a.key & 1u) | (KRON ? 2u : 0u) | ((unsigned)(nbr - 1) << 4);
    it.nblocks = a.nblocks + z.nblocks;
    std::snprintf(it.label, sizeof(it.label), "k_ttm_duo<%s, %d, %s>", (a.key & 1u) ? "asi::bf16_t" : "float", nbr, KRON ? "true" : "false");
    std::snprintf(it.role, sizeof(it.role), "%s+%s", a.role, z.role);
    it.bytes = a.bytes + z.bytes; it.flops = a.flops + z.flops;
    static_assert(sizeof(J) <= kItemArgMax, "argument block");
    std::memcpy(it.arg, &jb, sizeof(jb));
    *out = it;
    return true;
}
bool make_ttm_duo(const Item& a, const Item& z, Item* out) {
    const bool kron = z.kind == IT_TTM && (z.key & 0x600fu) == (2u | 4u);     // fp32, last mode, Kronecker, tiled, chunks of 32
    if (!kron && z.kind != IT_Z_PLANES) return false;
    if (a.kind == IT_TTM_STREAM) return !kron && make_ttm_stream_duo(a, z, out);
    if (a.kind != IT_TTM || (a.key & 0xc00eu) != 0u) return false;       // not last mode, plain, tiled, chunks of 32
    return kron ? put_ttm_duo<true>(a, z, out) : put_ttm_duo<false>(a, z, out);
}

template <typename T, bool KRON>
static hipError_t launch_duo(const Item* const* items, int n, int nbr, hipStream_t st) {
    Batch<TtmDuoJob<KRON>> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    switch (nbr) {
        case 1: hipLaunchKernelGGL((k_ttm_duo<T, 1, KRON>), grid, 256, 0, st, b); break;
        case 2: hipLaunchKernelGGL((k_ttm_duo<T, 2, KRON>), grid, 256, 0, st, b); break;
        case 3: hipLaunchKernelGGL((k_ttm_duo<T, 3, KRON>), grid, 256, 0, st, b); break;
        default: hipLaunchKernelGGL((k_ttm_duo<T, 4, KRON>), grid, 256, 0, st, b); break;
    }
    return hipGetLastError();
}
hipError_t launch_ttm_duo_items(const Item* const* items, int n, hipStream_t st, char* label_out) {
    const bool bf16 = items[0]->key & 1u, kron = items[0]->key & 2u;
    int nbr = 1;
    for (int j = 0; j < n; ++j) {
        const int nj = (int)((items[j]->key >> 4) & 7u) + 1;
        nbr = nj > nbr ? nj : nbr;
    }
    if (label_out) std::snprintf(label_out, 96, "k_ttm_duo<%s, %d, %s>", bf16 ? "asi::bf16_t" : "float", nbr, kron ? "true" : "false");
    if (kron) return bf16 ? launch_duo<bf16_t, true>(items, n, nbr, st) : launch_duo<float, true>(items, n, nbr, st);
    return bf16 ? launch_duo<bf16_t, false>(items, n, nbr, st) : launch_duo<float, false>(items, n, nbr, st);
}

hipError_t launch_ttm_expand_items(const Item* const* items, int n, hipStream_t st) {
    Batch<TtmJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ttm_expand, grid, 256, 0, st, b);
    return hipGetLastError();
}

hipError_t launch_ttm_items(const Item* const* items, int n, hipStream_t st, char* label_out) {
    Batch<TtmJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const unsigned key = items[0]->key;
    const bool bf16 = key & 1u, last = key & 2u, kron = key & 4u, ksplit = key & 8u;
    const bool kc64 = key & 0x4000u, contig = key & 0x40000u;
    const int cb = 1 + (int)((key >> 16) & 1u), nw = (key >> 17) & 1u ? 4 : 8;
    if (key & 0x8000u) {             // very short mode: one instantiation per bound on n
        int nmax = 8;
        for (int j = 0; j < n; ++j) {
            TtmJob tj;
            std::memcpy(&tj, items[j]->arg, sizeof(tj));
            if (tj.n > 8) nmax = 16;
        }
        if (label_out) std::snprintf(label_out, 96, "k_ttm_thin<%s, %d>", bf16 ? "asi::bf16_t" : "float", nmax);
        if (!bf16) { if (nmax == 8) hipLaunchKernelGGL((k_ttm_thin<float, 8>), grid, 256, 0, st, b); else hipLaunchKernelGGL((k_ttm_thin<float, 16>), grid, 256, 0, st, b); }
        else { if (nmax == 8) hipLaunchKernelGGL((k_ttm_thin<bf16_t, 8>), grid, 256, 0, st, b); else hipLaunchKernelGGL((k_ttm_thin<bf16_t, 16>), grid, 256, 0, st, b); }
        return hipGetLastError();
    }
    // the instantiation with the most output blocks serves every item
    int nbr = 1;
    for (int j = 0; j < n; ++j) {
        const int nj = (int)((items[j]->key >> 4) & 7u) + 1;
        nbr = nj > nbr ? nj : nbr;
    }
    if (label_out) {
        const char* tn = bf16 ? "asi::bf16_t" : "float";
        if (ksplit) std::snprintf(label_out, 96, "k_ttm_ksplit<%s, %d, %d, %s, %d>", tn, nbr, cb, contig ? "true" : "false", nw);
        else std::snprintf(label_out, 96, "k_ttm_mfma<%s, %s, %d, %d>", tn, last ? "true" : "false", nbr, kron ? (kc64 ? 2 : 1) : (kc64 ? 3 : 0));
    }
    if (ksplit) {
        if (!bf16) {
            switch (nbr) {
                case 1: return launch_split<float, 1>(cb, nw, contig, b, grid, st);
                case 2: return launch_split<float, 2>(cb, nw, contig, b, grid, st);
                case 3: return launch_split<float, 3>(cb, nw, contig, b, grid, st);
                default: return launch_split<float, 4>(cb, nw, contig, b, grid, st);
            }
        } else {
            switch (nbr) {
                case 1: return launch_split<bf16_t, 1>(cb, nw, contig, b, grid, st);
                case 2: return launch_split<bf16_t, 2>(cb, nw, contig, b, grid, st);
                case 3: return launch_split<bf16_t, 3>(cb, nw, contig, b, grid, st);
                default: return launch_split<bf16_t, 4>(cb, nw, contig, b, grid, st);
            }
        }
    } else if (kron) {           // always LASTMODE
        if (!bf16) { if (kc64) launch_tiled<float, true, 2>(nbr, b, grid, st); else launch_tiled<float, true, 1>(nbr, b, grid, st); }
        else { if (kc64) launch_tiled<bf16_t, true, 2>(nbr, b, grid, st); else launch_tiled<bf16_t, true, 1>(nbr, b, grid, st); }
    } else if (!bf16) {
        if (last && kc64) launch_tiled<float, true, 3>(nbr, b, grid, st);
        else if (last) launch_tiled<float, true, 0>(nbr, b, grid, st);
        else launch_tiled<float, false, 0>(nbr, b, grid, st);
    } else {
        if (last && kc64) launch_tiled<bf16_t, true, 3>(nbr, b, grid, st);
        else if (last) launch_tiled<bf16_t, true, 0>(nbr, b, grid, st);
        else launch_tiled<bf16_t, false, 0>(nbr, b, grid, st);
    }
    return hipGetLastError();
}

}  // namespace asi
