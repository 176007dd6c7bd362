// Subspace-iteration step of the LAST TWO modes of a tensor seen as (planes, rows, cols), planes of up to 64 x 64: the H
// and W modes of a conv activation, both from one read of it, through their Gram matrices.
//
// Alg. 1 asks for P = A_m (A_m^T U_prev) = (A_m A_m^T) U_prev.  For one plane X (rows x cols)
//     mode H:   G_H += X X^T   (rows x rows),      P_H = G_H U_H
//     mode W:   G_W += X^T X   (cols x cols),      P_W = G_W U_W
// so the planes only feed the two Gram matrices, in fp64 (products of fp32 values are exact there), and U_prev is
// multiplied once per workgroup at the end.  Against the two products per plane (V on the fp32 MFMA, P on the fp64 MFMA;
// the form this kernel had before) a 64 x 64 plane costs 160 instead of 192 fp64-MFMA units a mode at rank 32, the padding
// of ranks and of the last column block is gone (56 x 56 at rank 24: 140 instead of 192), both operands of a product
// are the same registers, V is never rounded to fp32, and nothing but the operands has to be in LDS.
//
// A tile is a run of whole planes, contiguous in memory, copied to LDS as it is (16 bytes per lane and instruction
// straight from memory to LDS, no register and no vector instruction on the way) while the previous tile is multiplied:
// two buffers, one wait per tile.  Eight waves: wave w < 4 accumulates G_H of planes w, w + 4, .., wave w + 4 the G_W of
// the same planes, one of each on every SIMD.  Operand of K slot lg: lane (lg, ll) holds element (M = 16 mb + ll, K), for
// the A and the B side alike; K slot (s, lg) of a block of 16 stands for index 16 kb + 4 lg + s, of a last block of
// 4 nst or fewer for 16 kb + nst lg + s.  Rows past the plane read what lies behind it and only reach rows and columns of G
// that are dropped; a K index past the plane is masked.  LDS bank conflicts of the unpadded rows (up to 4-way) do not
// matter: a read feeds at least 256 cycles of the matrix pipe.
//
// Bound: fp64 MFMA for planes beyond 32 x 32 (under this load the clock is 2.1 GHz, the pipe's rate 67 TFLOP/s), memory below.
// 4096 planes of 56 x 56 (rank 24) 62.9 -> 52.3 us: 7 us to the first product and after the last (launch, first tile, sum
// over the waves, the product with U_prev), 10.7 us a tile of which the products alone need 8.5.  2048 of 64 x 64 (rank 32)
// 37.0 -> 35.4, 16384 of 14 x 14 (rank 7) 17.2 -> 11.9, 1079 of 45 x 37 16.4 -> 15.8.
#include "asi_gram_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

constexpr int PN_NT = 512;                 // eight waves

struct PlanesJob {
    const void* X;
    long long planes, ntiles;
    const float* U[2];       // (rows, r[0]) and (cols, r[1])
    double* part[2];         // (nwg, rows, r[0]) and (nwg, cols, r[1])
    int rows, cols, r[2];
    int pt;                  // planes per tile
    int buf;                 // bytes of one LDS buffer
    int lds;                 // bytes of LDS a launch needs
    int nwg;
    int32_t* zero;           // nullable: `nzero` int32 the kernel clears
    int nzero;
};

extern __shared__ __align__(16) unsigned char pn_raw[];

// Gram products of one plane for one mode.  H: M runs over the rows (stride cols), K over the columns (stride 1); W the
// other way.  All NB blocks of M are multiplied (a plane that is shorter one way than the other reads on into what follows
// it and those blocks are dropped): a test per block costs a branch per product.
template <typename T, int NB, bool H>
__device__ __forceinline__ void plane_gram(const T* xp, int cols, int k, bool vec, int lg, int ll, v4d* acc) {
    const T* base = xp + (H ? ll * cols : ll);
    const int mstep = H ? 16 * cols : 16;              // elements between blocks of the M index
    const int nfull = k >> 4, rem = k & 15;
#pragma unroll 1
    for (int kb = 0; kb < nfull; ++kb) {
        double d[NB][4];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) {
            float x[4];
            const T* q = base + mb * mstep;
            if constexpr (H) {
                read4(q + 16 * kb + 4 * lg, vec, x);
            } else {
#pragma unroll
                for (int s = 0; s < 4; ++s) x[s] = to_f32(q[(16 * kb + 4 * lg + s) * cols]);
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) d[mb][s] = (double)x[s];
        }
#pragma unroll
        for (int s = 0; s < 4; ++s) gram_step<NB>(d, s, acc);
    }
    if (rem) {
        const int nst = (rem + 3) >> 2;                // K steps of the last block
        double d[NB][4];
#pragma unroll
        for (int mb = 0; mb < NB; ++mb)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int kk = nst * lg + (s < nst ? s : 0);
                const float x = to_f32(base[mb * mstep + (H ? 16 * nfull + kk : (16 * nfull + kk) * cols)]);
                d[mb][s] = kk < rem ? (double)x : 0.0;
            }
        gram_step<NB>(d, 0, acc);
        if (nst > 1) gram_step<NB>(d, 1, acc);
        if (nst > 2) gram_step<NB>(d, 2, acc);
        if (nst > 3) gram_step<NB>(d, 3, acc);
    }
}

template <typename T, int NB, bool DMA>
__global__ __launch_bounds__(PN_NT, NB <= 2 ? 4 : 2) void k_subspace_planes(Batch<PlanesJob> bt) {
    constexpr int NP = gram_blocks<NB>();              // blocks of G on and above the diagonal
    constexpr int NA = NB == 1 ? 2 : 1;                // one block: planes alternate between two accumulators
    int lb;
    const PlanesJob& jb = bt.job[locate(bt, &lb)];
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const int rows = jb.rows, cols = jb.cols, pe = rows * cols, pt = jb.pt, buf = jb.buf;
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int role = wv >> 2, slot = wv & 3;           // role 0: mode H (rows), role 1: mode W (cols)
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;

    auto fetch = [&](long long t, int b) __attribute__((always_inline)) {
        const long long p0 = t * pt;
        const int np = (int)(jb.planes - p0 < pt ? jb.planes - p0 : pt);
        const int elems = np * pe;
        const T* src = X + p0 * pe;
        unsigned char* dst = pn_raw + b * buf;
        if constexpr (DMA) {
            const int bytes = elems * (int)sizeof(T), npc = bytes >> 4;
            for (int j = 0; j < npc; j += PN_NT) {     // a wave's 64 lanes fill 1 KB of LDS per instruction
                const int pc = j + tid;
                if (pc < npc) copy16_to_lds(src, bytes, pc * 16, dst + (j + 64 * wv) * 16);
            }
            const int tail = npc * (16 / (int)sizeof(T)) + tid;        // what is left of the tensor's last plane (under 16 bytes)
            if (tail < elems) reinterpret_cast<T*>(dst)[tail] = src[tail];
        } else {
            for (int e0 = 0; e0 < elems; e0 += 8 * PN_NT) {            // element by element: a tensor aligned to its element only
                T v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = e0 + u * PN_NT + tid;
                    v[u] = src[e < elems ? e : 0];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = e0 + u * PN_NT + tid;
                    if (e < elems) reinterpret_cast<T*>(dst)[e] = v[u];
                }
            }
        }
    };
    v4d acc[NA][NP];
#pragma unroll
    for (int a = 0; a < NA; ++a)
#pragma unroll
        for (int p = 0; p < NP; ++p) acc[a][p] = (v4d){0.0, 0.0, 0.0, 0.0};
    const bool vec = (cols & 3) == 0;                  // (planes then start at a multiple of four elements, too)

    if (lb < jb.ntiles) fetch(lb, 0);
    int b = 0;
    for (long long t = lb; t < jb.ntiles; t += jb.nwg, b ^= 1) {
        if constexpr (DMA) wait_copies_and_sync<0>();
        __syncthreads();                               // tile t is in LDS; the other buffer is no longer read
        if (t + jb.nwg < jb.ntiles) fetch(t + jb.nwg, b ^ 1);
        const long long p0 = t * pt;
        const int np = (int)(jb.planes - p0 < pt ? jb.planes - p0 : pt);
        const T* xb = reinterpret_cast<const T*>(pn_raw + b * buf);
        if (role == 0) {
            for (int p = slot; p < np; p += 4 * NA) {
                plane_gram<T, NB, true>(xb + p * pe, cols, cols, vec, lg, ll, acc[0]);
                if (NA == 2 && p + 4 < np) plane_gram<T, NB, true>(xb + (p + 4) * pe, cols, cols, vec, lg, ll, acc[NA - 1]);
            }
        } else {
            for (int p = slot; p < np; p += 4 * NA) {
                plane_gram<T, NB, false>(xb + p * pe, cols, rows, vec, lg, ll, acc[0]);
                if (NA == 2 && p + 4 < np) plane_gram<T, NB, false>(xb + (p + 4) * pe, cols, rows, vec, lg, ll, acc[NA - 1]);
            }
        }
    }
    if (NA == 2)
#pragma unroll
        for (int p = 0; p < NP; ++p) acc[0][p] += acc[NA - 1][p];

    // Sum of the four waves of a mode, both modes at once: waves 2 and 3 hand their blocks to waves 0 and 1, wave 1 its sum to
    // wave 0 (fixed order), wave 0 leaves G in LDS; then the four multiply by U_prev.
    double* red = reinterpret_cast<double*>(pn_raw);   // [2 modes][2][NP][256]
    const int n = role ? cols : rows, r = jb.r[role];
    const float* __restrict__ U = jb.U[role];
    float u[NB][4];
    gram_load_u<NB>(U, n, r, slot, lane, u);
    double* mine = red + (2 * role + (slot & 1)) * NP * 256;
    __syncthreads();                                   // the tiles are no longer read
    if (slot >= 2) gram_put<NB>(acc[0], mine, lane);
    __syncthreads();
    if (slot < 2) gram_add<NB>(acc[0], mine, lane);
    if (slot == 1) gram_put<NB>(acc[0], mine, lane);
    __syncthreads();
    if (slot == 0) {
        gram_add<NB>(acc[0], mine + NP * 256, lane);
        gram_put<NB>(acc[0], mine, lane);
    }
    __syncthreads();
    gram_times_u<NB, 4>(red + 2 * role * NP * 256, U, n, r, jb.part[role] + (long long)lb * n * r, slot, lane, u);
}

// ---- planes of up to 8 x 8 (7 x 7 maps) --------------------------------------------------------------------
// The same Gram matrices with TWO planes stacked in the 16 rows of an operand: the two 8 x 8 blocks on the diagonal of the 16 x 16
// result are theirs, what lies off it is dropped, and a mode of a pair of planes costs two MFMAs (K slot (s, lg) is index 2 lg + s), a
// quarter of what one plane a block of 16 x 16 x 16 takes.  Tiles of 16 KB go through a ring of four buffers, three of them on their
// way; what a tile does not fill arrives as zeros, so that an odd last plane has a partner of zeros.
// 122880 planes of 7 x 7 at rank 6 (24 MB): 128 cycles of MFMA a plane, 6.5 us; 19.8 -> 17.0 us against a thread per plane and mode on the
// vector ALU, three batched layers of 32768 planes 21.8 -> 17.2.
constexpr int TY_BUF = 16384, TY_RING = 4, TY_COPIES = TY_BUF / (16 * PN_NT);
struct TinyJob {
    const void* X;
    long long planes, ntiles;
    const float* U[2];    // (rows, r[0]) and (cols, r[1])
    double* part[2];      // (nwg, rows, r[0]) and (nwg, cols, r[1])
    int rows, cols, r[2];
    int pt;               // planes per tile, a multiple of eight
    int nwg;
};

template <typename T, bool DMA>
__global__ __launch_bounds__(PN_NT, 4) void k_subspace_tiny(Batch<TinyJob> bt) {
    int lb;
    const TinyJob& jb = bt.job[locate(bt, &lb)];
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const int rows = jb.rows, cols = jb.cols, pe = rows * cols, pt = jb.pt;
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int role = wv >> 2, slot = wv & 3;           // role 0: mode H (rows), role 1: mode W (cols)
    auto elems_of = [&](long long t) __attribute__((always_inline)) {
        const long long left = jb.planes - t * pt;
        return left <= 0 ? 0 : (int)(left < pt ? left : pt) * pe;
    };
    auto fetch = [&](long long t, int b) __attribute__((always_inline)) {
        const int elems = elems_of(t);
        const T* src = X + (elems ? t * pt * pe : 0);
        unsigned char* dst = pn_raw + b * TY_BUF;
        if constexpr (DMA) {
            const int whole = elems * (int)sizeof(T) & ~15;
#pragma unroll
            for (int u = 0; u < TY_COPIES; ++u)
                copy16_to_lds(src, whole, (u * PN_NT + tid) * 16, dst + (u * PN_NT + 64 * wv) * 16);
        } else {
            constexpr int PER = TY_BUF / (int)sizeof(T) / PN_NT;
            for (int u0 = 0; u0 < PER; u0 += 8) {      // element by element: a tensor aligned to its element only
                T v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = (u0 + u) * PN_NT + tid;
                    v[u] = src[e < elems ? e : 0];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int e = (u0 + u) * PN_NT + tid;
                    reinterpret_cast<T*>(dst)[e] = e < elems ? v[u] : T();
                }
            }
        }
    };
    // this lane's two elements of a pair of planes: plane ll / 8, index ll % 8 of the mode, indices 2 lg and 2 lg + 1 of the other
    const int k = role == 0 ? cols : rows, ks = role == 0 ? 1 : cols, ms = role == 0 ? cols : 1;
    const bool in0 = 2 * lg < k, in1 = 2 * lg + 1 < k;
    const int o0 = (ll >> 3) * pe + (ll & 7) * ms + (in0 ? 2 * lg : 0) * ks, o1 = (ll >> 3) * pe + (ll & 7) * ms + (in1 ? 2 * lg + 1 : 0) * ks;
    v4d acc[2] = {{0.0, 0.0, 0.0, 0.0}, {0.0, 0.0, 0.0, 0.0}};

    constexpr int AHEAD = DMA ? TY_RING - 1 : 1;       // tiles on their way
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) fetch(lb + (long long)u * jb.nwg, u);
    int b = 0;
    for (long long t = lb; t < jb.ntiles; t += jb.nwg) {
        if constexpr (DMA) wait_copies_and_sync<(TY_RING - 2) * TY_COPIES>();
        else __syncthreads();                          // tile t is in LDS; the buffer of the tile before is no longer read
        fetch(t + (long long)AHEAD * jb.nwg, (b + AHEAD) & (TY_RING - 1));
        const int elems = elems_of(t), np = elems / pe;
        T* xb = reinterpret_cast<T*>(pn_raw + b * TY_BUF);
        if (DMA && ((elems * (int)sizeof(T)) & 15)) {  // uniform: the end of the tensor, under 16 bytes past the last whole piece
            const int e = (elems * (int)sizeof(T) & ~15) / (int)sizeof(T) + tid;
            if (e < elems) xb[e] = X[t * pt * pe + e];
            __syncthreads();
        }
        const T* q = xb + 2 * slot * pe;
        const int pairs = ((np + 1) / 2 - slot + 3) / 4;        // of this wave: pairs slot, slot + 4, ..
        int i = 0;
        for (; i + 1 < pairs; i += 2) {
            float x[4];
            x[0] = to_f32(q[o0]); x[1] = to_f32(q[o1]); x[2] = to_f32(q[8 * pe + o0]); x[3] = to_f32(q[8 * pe + o1]);
            const double d0 = in0 ? (double)x[0] : 0.0, d1 = in1 ? (double)x[1] : 0.0, d2 = in0 ? (double)x[2] : 0.0, d3 = in1 ? (double)x[3] : 0.0;
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d0, d0, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d2, d2, acc[1], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d1, d1, acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(d3, d3, acc[1], 0, 0, 0);
            q += 16 * pe;
        }
        if (i < pairs) {
            const float x0 = to_f32(q[o0]), x1 = to_f32(q[o1]);
            const double d0 = in0 ? (double)x0 : 0.0, d1 = in1 ? (double)x1 : 0.0;
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d0, d0, acc[0], 0, 0, 0);
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(d1, d1, acc[0], 0, 0, 0);
        }
        b = (b + 1) & (TY_RING - 1);
    }
    acc[0] += acc[1];
    if constexpr (DMA) wait_copies_and_sync<0>();      // (the last copies write zeros into buffers that the sums take over)

    // the four waves of a mode, both modes at once, as in k_subspace_planes; then the two diagonal blocks
    double* red = reinterpret_cast<double*>(pn_raw);   // [2 modes][2][256]
    const int n = role ? cols : rows, r = jb.r[role];
    const float* __restrict__ U = jb.U[role];
    float u[1][4];
    gram_load_u<1>(U, n, r, slot, lane, u);
    double* mine = red + (2 * role + (slot & 1)) * 256;
    __syncthreads();                                   // the tiles are no longer read
    if (slot >= 2) gram_put<1>(&acc[0], mine, lane);
    __syncthreads();
    if (slot < 2) gram_add<1>(&acc[0], mine, lane);
    if (slot == 1) gram_put<1>(&acc[0], mine, lane);
    __syncthreads();
    if (slot == 0) {
        gram_add<1>(&acc[0], mine + 256, lane);
        gram_put<1>(&acc[0], mine, lane);
    }
    __syncthreads();
    if (tid < 128) {
        const int i = (tid >> 3) & 7, j = tid & 7;     // element (i, j) at (i / 4) 64 + (i % 4) 16 + j
        double* g = red + 2 * (tid >> 6) * 256 + (i >> 2) * 64 + (i & 3) * 16 + j;
        *g += g[128 + 8];
    }
    __syncthreads();
    gram_times_u<1, 4>(red + 2 * role * 256, U, n, r, jb.part[role] + (long long)lb * n * r, slot, lane, u);
}

bool subspace_tiny_supported(int rows, int cols, int r_rows, int r_cols) {
    return rows <= 8 && cols <= 8 && r_rows <= rows && r_cols <= cols;
}
static int tiny_pt(DType xt, int rows, int cols) {
    // (an operand's rows past a plane reach up to 63 elements past the last one: they stay in the buffer)
    const int pt = (TY_BUF - 256) / (rows * cols * (xt == F32 ? 4 : 2)) / 8 * 8;
    return pt > 512 ? 512 : pt;
}
// two workgroups per CU are resident, and every one walks the same number of tiles
int subspace_tiny_nwg(DType xt, long long planes, int rows, int cols) {
    const long long pt = tiny_pt(xt, rows, cols), ntiles = (planes + pt - 1) / pt, per = (ntiles + 511) / 512;
    return (int)((ntiles + per - 1) / per);
}
// key: [0] bf16, [1] memory-to-LDS copies
bool make_subspace_tiny(DType xt, const void* X, long long planes, int rows, int cols, const float* U_rows, int r_rows,
                        double* part_rows, const float* U_cols, int r_cols, double* part_cols, int nwg, Item* out) {
    if (!subspace_tiny_supported(rows, cols, r_rows, r_cols) || !X || !U_rows || !U_cols || !part_rows || !part_cols)
        return false;
    if (planes < 1 || rows < 1 || cols < 1 || nwg != subspace_tiny_nwg(xt, planes, rows, cols)) return false;
    TinyJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.planes = planes; jb.pt = tiny_pt(xt, rows, cols); jb.ntiles = (planes + jb.pt - 1) / jb.pt;
    jb.U[0] = U_rows; jb.U[1] = U_cols; jb.part[0] = part_rows; jb.part[1] = part_cols;
    jb.rows = rows; jb.cols = cols; jb.r[0] = r_rows; jb.r[1] = r_cols; jb.nwg = nwg;
    *out = Item();
    out->kind = IT_TINY;
    const bool dma = reinterpret_cast<uintptr_t>(X) % 16 == 0;       // (a tile of a multiple of eight planes is a multiple of 16 bytes)
    out->key = (xt == BF16 ? 1u : 0u) | (dma ? 2u : 0u);
    out->nblocks = nwg;
    std::snprintf(out->label, sizeof(out->label), "k_subspace_tiny<%s, %s>", xt == F32 ? "float" : "asi::bf16_t", dma ? "true" : "false");
    static_assert(sizeof(TinyJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}
hipError_t launch_tiny_items(const Item* const* items, int n, hipStream_t st) {
    Batch<TinyJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    constexpr size_t lds = TY_RING * TY_BUF;
    switch (items[0]->key) {
        case 0: hipLaunchKernelGGL((k_subspace_tiny<float, false>), grid, PN_NT, lds, st, b); break;
        case 1: hipLaunchKernelGGL((k_subspace_tiny<bf16_t, false>), grid, PN_NT, lds, st, b); break;
        case 2: hipLaunchKernelGGL((k_subspace_tiny<float, true>), grid, PN_NT, lds, st, b); break;
        case 3: hipLaunchKernelGGL((k_subspace_tiny<bf16_t, true>), grid, PN_NT, lds, st, b); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---- host side ---------------------------------------------------------------------------------
bool subspace_planes_supported(long long planes, int rows, int cols, int r_rows, int r_cols) {
    if (planes < 1 || rows < 1 || rows > 64 || cols < 1 || cols > 64) return false;
    return r_rows >= 1 && r_cols >= 1 && r_rows <= rows && r_cols <= cols;
}
static int planes_nb(int rows, int cols) { return (std::max(rows, cols) + 15) / 16; }
// Planes per tile: a wave takes every fourth, so at least four (eight for bf16, whose tiles then start at 16 bytes whatever
// the plane); more for small planes, up to ~32 KB, as long as every CU still gets a tile.
static int planes_pt(DType xt, long long planes, int rows, int cols) {
    const int least = xt == F32 ? 4 : (rows * cols * 2 % 4 == 0 ? 4 : 8);
    const long long pb = (long long)rows * cols * (xt == F32 ? 4 : 2);
    int pt = least;
    while (2 * pt * pb <= 32768 && planes >= 256LL * 2 * pt) pt *= 2;
    return pt;
}
int subspace_planes_nwg(DType xt, long long planes, int rows, int cols) {
    const int pt = planes_pt(xt, planes, rows, cols);
    const long long ntiles = (planes + pt - 1) / pt;
    // resident workgroups: one per CU beyond 32 x 32 (accumulators), else two; every one walks the same number of tiles
    const long long most = planes_nb(rows, cols) > 2 ? 256 : 512, per = (ntiles + most - 1) / most;
    return (int)((ntiles + per - 1) / per);
}

// key: [0] bf16, [1] memory-to-LDS copies, [4..6] NB
bool make_subspace_planes(DType xt, const void* X, long long planes, int rows, int cols, const float* U_rows, int r_rows,
                          double* part_rows, const float* U_cols, int r_cols, double* part_cols, int nwg, int32_t* zero,
                          int nzero, Item* out) {
    if (!subspace_planes_supported(planes, rows, cols, r_rows, r_cols) || !X || !U_rows || !U_cols || !part_rows || !part_cols)
        return false;
    if (nzero < 0 || nzero > 256 || nwg != subspace_planes_nwg(xt, planes, rows, cols)) return false;
    PlanesJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.planes = planes; jb.pt = planes_pt(xt, planes, rows, cols); jb.ntiles = (planes + jb.pt - 1) / jb.pt;
    jb.U[0] = U_rows; jb.U[1] = U_cols; jb.part[0] = part_rows; jb.part[1] = part_cols;
    jb.rows = rows; jb.cols = cols; jb.r[0] = r_rows; jb.r[1] = r_cols; jb.nwg = nwg;
    jb.zero = zero; jb.nzero = zero ? nzero : 0;
    const int es = xt == F32 ? 4 : 2, nb = planes_nb(rows, cols);
    jb.buf = (jb.pt * rows * cols * es + 15) / 16 * 16;
    *out = Item();
    out->kind = IT_PLANES;
    const bool dma = reinterpret_cast<uintptr_t>(X) % 16 == 0 && (jb.pt * rows * cols * es) % 16 == 0;
    out->key = (xt == BF16 ? 1u : 0u) | (dma ? 2u : 0u) | ((unsigned)nb << 4);
    out->nblocks = nwg;
    // what a launch needs: two buffers and the reach of the reads past the last plane, or the sums of the end
    const int c16 = (cols + 15) / 16 * 16, r16 = (rows + 15) / 16 * 16;
    const int reach = std::max((16 * nb - 1) * cols + c16, (r16 - 1) * cols + 16 * nb) * es;      // from a plane's first element
    jb.lds = std::max(2 * jb.buf + reach - rows * cols * es + 16, 4 * (nb * (nb + 1) / 2) * 256 * 8);
    std::snprintf(out->label, sizeof(out->label), "k_subspace_planes<%s, %d, %s>", xt == F32 ? "float" : "asi::bf16_t", nb,
                  dma ? "true" : "false");
    static_assert(sizeof(PlanesJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

template <typename T, int NB, bool DMA>
static hipError_t launch_planes_t(const Batch<PlanesJob>& b, dim3 grid, int lds, hipStream_t st) {
    if (lds > 65536) {
        static LdsAllowed allowed;
        const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_subspace_planes<T, NB, DMA>), 160 * 1024, allowed);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_subspace_planes<T, NB, DMA>), grid, PN_NT, lds, st, b);
    return hipGetLastError();
}
template <typename T, bool DMA>
static hipError_t launch_planes_nb(const Batch<PlanesJob>& b, dim3 grid, int nb, int lds, hipStream_t st) {
    switch (nb) {
        case 1: return launch_planes_t<T, 1, DMA>(b, grid, lds, st);
        case 2: return launch_planes_t<T, 2, DMA>(b, grid, lds, st);
        case 3: return launch_planes_t<T, 3, DMA>(b, grid, lds, st);
        case 4: return launch_planes_t<T, 4, DMA>(b, grid, lds, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_planes_items(const Item* const* items, int n, hipStream_t st) {
    Batch<PlanesJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    int lds = 0;
    for (int j = 0; j < n; ++j) lds = std::max(lds, b.job[j].lds);
    const unsigned key = items[0]->key;
    const int nb = (int)((key >> 4) & 7u);
    if (key & 1u) return (key & 2u) ? launch_planes_nb<bf16_t, true>(b, grid, nb, lds, st) : launch_planes_nb<bf16_t, false>(b, grid, nb, lds, st);
    return (key & 2u) ? launch_planes_nb<float, true>(b, grid, nb, lds, st) : launch_planes_nb<float, false>(b, grid, nb, lds, st);
}

}  // namespace asi
