// Kernel body of the Gram form of a subspace step (asi_gram.hip), on its own so that a launch can do several modes' steps.
#pragma once
#include "asi_gram_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"

namespace asi {

constexpr int SG_NT = 512, SG_NW = SG_NT / 64;
constexpr int SG_MAX_WG = 256;             // one workgroup per CU, each walking several tiles
template <int NB> constexpr int sg_row_bytes() { return NB == 1 ? 1024 : 512; }
template <int NB> constexpr int sg_buf_bytes() { return 16 * (NB <= 2 ? NB : 4) * sg_row_bytes<NB>(); }     // 16, 16, 32, 32 KB
template <int NB> constexpr int sg_nbuf() { return NB <= 2 ? 6 : 4; }

template <int NB> constexpr int sg_lds_bytes() {
    const int ring = sg_nbuf<NB>() * sg_buf_bytes<NB>(), sums = 4 * gram_blocks<NB>() * 256 * 8;
    return ring > sums ? ring : sums;
}

struct GramJob {
    const void* X;       // (outer, n, inner)
    const float* U;      // (n, r) previous factor
    double* part;        // (nwg, n, r) partial sums of P
    long long outer, inner;
    int tiles_per_o, ntiles;
    int n, r, nwg;
    int S;               // n <= 8: S = 2 (n <= 4: 4) column ranges of a tile are stacked in the 16 LDS rows
    int32_t* zero;       // nullable: `nzero` int32 to clear
    int nzero;
};

extern __shared__ __align__(16) unsigned char sg_raw[];

// DMA: X starts 16-byte aligned, rows are a multiple of 16 bytes long and a slice is below 2 GiB; otherwise single elements
// through registers.
template <typename T, int NB, bool DMA>
__device__ __forceinline__ void subspace_gram(const GramJob& jb, int lb) {
    constexpr int RB = sg_row_bytes<NB>(), TC = RB / (int)sizeof(T), BUF = sg_buf_bytes<NB>(), NBUF = sg_nbuf<NB>();
    constexpr int PPR = RB / 16, NP = gram_blocks<NB>();
    constexpr int NL = BUF / 16 / SG_NT;                   // copies per thread and tile
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = jb.n, r = jb.r, S = NB == 1 ? jb.S : 1, rows = S * n;
    const long long inner = jb.inner;
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;

    auto origin = [&](int tile, int* o, long long* j0, int* vc) __attribute__((always_inline)) {
        *o = (unsigned)tile / (unsigned)jb.tiles_per_o;
        *j0 = (long long)(tile - *o * jb.tiles_per_o) * (TC * S);
        *vc = (int)(inner - *j0 < TC * S ? inner - *j0 : TC * S);
    };
    // ---- copies: piece u * SG_NT + tid of a tile is LDS slot (row, slot) = global piece slot ^ (row % 16) of the row
    constexpr int FAR = 0x7ffffff0;                        // past any descriptor's extent: the copy writes zeros
    int goff[DMA ? NL : 1], gcol[DMA ? NL : 1];            // byte offset from the tile's first element; its column range
    if constexpr (DMA) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            const int pc = u * SG_NT + tid, row = pc / PPR, cp = (pc % PPR) ^ (row & 15);
            const int sidx = S > 1 ? row / n : 0, i = row - sidx * n;
            gcol[u] = row < rows ? (sidx * TC) * (int)sizeof(T) + 16 * cp : FAR;
            goff[u] = (int)(i * inner * (int)sizeof(T)) + (sidx * TC) * (int)sizeof(T) + 16 * cp;
        }
    }
    auto copy = [&](int tile, int b) __attribute__((always_inline)) {
        int o = 0, vc = 0;
        long long j0 = 0;
        if (tile < jb.ntiles) origin(tile, &o, &j0, &vc);  // (past the last tile: nothing is valid, zeros)
        const T* base = X + (long long)o * n * inner + j0;
        const int extent = (int)((n * inner - j0) * (long long)sizeof(T));
#pragma unroll
        for (int u = 0; u < NL; ++u)
            copy16_to_lds(base, extent, gcol[u] < vc * (int)sizeof(T) ? goff[u] : FAR, sg_raw + b * BUF + (u * SG_NT + 64 * wave) * 16);
    };
    // ---- element-wise form: a tile waits in registers while the one before it is multiplied
    constexpr int NE = BUF / (int)sizeof(T) / SG_NT;
    T pre[DMA ? 1 : NE];
    auto fetch = [&](int tile) __attribute__((always_inline)) {
        int o, vc;
        long long j0;
        origin(tile, &o, &j0, &vc);
        const T* base = X + (long long)o * n * inner + j0;
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const int e = u * SG_NT + tid, row = e / TC, c = e % TC;
            const int sidx = S > 1 ? row / n : 0, i = row - sidx * n;
            const bool ok = row < rows && sidx * TC + c < vc;
            pre[DMA ? 0 : u] = base[ok ? i * inner + sidx * TC + c : 0];
        }
    };
    auto store = [&](int tile, int b) __attribute__((always_inline)) {
        int o, vc;
        long long j0;
        origin(tile, &o, &j0, &vc);
#pragma unroll
        for (int u = 0; u < NE; ++u) {
            const int e = u * SG_NT + tid, row = e / TC, c = e % TC, cb = c * (int)sizeof(T);
            const int sidx = S > 1 ? row / n : 0;
            const bool ok = row < rows && sidx * TC + c < vc;
            T z;
            memset(&z, 0, sizeof(z));
            *reinterpret_cast<T*>(sg_raw + b * BUF + row * RB + (((cb >> 4) ^ (row & 15)) << 4) + (cb & 15)) = ok ? pre[DMA ? 0 : u] : z;
        }
    };

    v4d acc[NP];
#pragma unroll
    for (int p = 0; p < NP; ++p) acc[p] = (v4d){0.0, 0.0, 0.0, 0.0};
    if constexpr (DMA) {
#pragma unroll
        for (int b = 0; b < NBUF - 1; ++b) copy(lb + b * jb.nwg, b);
    } else {
        if (lb < jb.ntiles) fetch(lb);
    }
    int b = 0;
    for (int tile = lb; tile < jb.ntiles; tile += jb.nwg) {
        if constexpr (DMA) {
            // this wave's copies of `tile` have landed (those of the NBUF - 2 tiles after it may be on their way), then
            // everybody's have; nobody reads the buffer of the tile before any more, which takes the next copy
            wait_copies_and_sync<NL * (NBUF - 2)>();
            copy(tile + (NBUF - 1) * jb.nwg, b == 0 ? NBUF - 1 : b - 1);
        } else {
            store(tile, b);
            __syncthreads();
            if (tile + jb.nwg < jb.ntiles) fetch(tile + jb.nwg);
        }
        const unsigned char* xs = sg_raw + b * BUF + ll * RB;
        for (int ch = wave; ch < TC / 16; ch += SG_NW) {
            double d[NB][4];
            const int off = sizeof(T) == 4 ? ((4 * ch + lg) ^ ll) * 16 : ((2 * ch + (lg >> 1)) ^ ll) * 16 + (lg & 1) * 8;
#pragma unroll
            for (int mb = 0; mb < NB; ++mb) {
                float x[4];
                read4(reinterpret_cast<const T*>(xs + 16 * mb * RB + off), true, x);
#pragma unroll
                for (int s = 0; s < 4; ++s) d[mb][s] = (double)x[s];
            }
#pragma unroll
            for (int s = 0; s < 4; ++s) gram_step<NB>(d, s, acc);
        }
        b = b + 1 == NBUF ? 0 : b + 1;
    }
    // G = sum over the eight waves (a tree, fixed order) in LDS, left in the first wave's place; then P = G U_prev
    float u[NB][4];
    gram_load_u<NB>(jb.U, n, r, wave, lane, u);            // on its way during the sums
    double* red = reinterpret_cast<double*>(sg_raw);       // [4][NP][256]
    double* mine = red + (wave & 3) * NP * 256;
    wait_copies_and_sync<0>();                             // the tiles are no longer read, the copies past the last one have landed
    __syncthreads();
    if (wave >= 4) gram_put<NB>(acc, mine, lane);
    __syncthreads();
    if (wave < 4) gram_add<NB>(acc, mine, lane);
    if (wave == 2 || wave == 3) gram_put<NB>(acc, mine, lane);
    __syncthreads();
    if (wave < 2) gram_add<NB>(acc, mine + 2 * NP * 256, lane);
    if (wave == 1) gram_put<NB>(acc, mine, lane);
    __syncthreads();
    if (wave == 0) {
        gram_add<NB>(acc, mine + NP * 256, lane);
        gram_put<NB>(acc, mine, lane);
    }
    __syncthreads();
    if (NB == 1 && S > 1) {                                // the ranges' Gram matrices lie along the diagonal of the block
        double g = 0.0;
        const int i = tid >> 4, k = tid & 15;
        if (i < n && k < n)
            for (int s = 0; s < S; ++s) {
                const int ii = s * n + i;
                g += red[(ii >> 2) * 64 + (ii & 3) * 16 + s * n + k];
            }
        __syncthreads();
        if (i < n && k < n) red[(i >> 2) * 64 + (i & 3) * 16 + k] = g;
        __syncthreads();
    }
    gram_times_u<NB, SG_NW>(red, jb.U, n, r, jb.part + (long long)lb * n * r, wave, lane, u);
}

}  // namespace asi
