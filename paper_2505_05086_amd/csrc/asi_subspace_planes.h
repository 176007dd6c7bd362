// Kernel bodies of the subspace steps of the last two modes (asi_planes.hip), on their own so that a launch can do several modes' steps.
#pragma once
#include "asi_gram_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"

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
__device__ __forceinline__ void subspace_planes(const PlanesJob& jb, int lb) {
    constexpr int NP = gram_blocks<NB>();              // blocks of G on and above the diagonal
    constexpr int NA = NB == 1 ? 2 : 1;                // one block: planes alternate between two accumulators
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
__device__ __forceinline__ void subspace_tiny(const TinyJob& jb, int lb) {
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

}  // namespace asi
