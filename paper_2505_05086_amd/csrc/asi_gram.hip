// Subspace-iteration step of a short mode with a long inner extent (the batch mode of an activation:
// n <= 64 indices, millions of unfolding columns) through the mode's Gram matrix.
//
// Alg. 1 asks for P = A_m V with V = A_m^T U_prev, i.e. P = (A_m A_m^T) U_prev.  For a short mode the
// n x n matrix G = A_m A_m^T is tiny, so the step is one pass over the activation that accumulates G
// and a product G U_prev at the end; V (columns x r) is never formed, not even in registers:
//     G[i][i'] = sum_c X[i][c] X[i'][c]      fp64 MFMA 16x16x4, both operands from ONE LDS read
//     P        = G U_prev                    fp64 MFMA, once per workgroup
// Products of fp32 (or bf16) values are exact in fp64 and the sums are carried in fp64, so P is at least
// as accurate as the two-product form (which rounds V to fp32 in between).
//
// A tile is the n rows of a range of columns, 16 or 32 KB.  The pass is bound by memory up to two row blocks (n <= 32), so
// what counts is how much of it is on its way: the tiles travel straight from memory to LDS, 16 bytes per lane and
// instruction, without registers or vector instructions, into a ring of buffers (16 KB each, six; 32 KB each, four) of
// which all but two are in flight while one is multiplied and one is being freed; one workgroup of eight waves per CU.
// What lies past the tensor's rows or past the columns of a slice is given an offset beyond the buffer descriptor's
// extent: the copy then writes zeros, so neither the copy nor the products have a test for it.  In LDS the 16-byte pieces
// of row i are permuted (piece p of the row sits at p ^ (i % 16)), which spreads the 16 rows an operand read touches over
// the banks.
//
// 32 entries over 401 K columns (51 MB) 24.4 -> 20.4 us, 64 over 605 K in bf16 (77 MB, bound by the fp64 MFMA: 40 us of
// products) 82 -> 71, 8 entries over 32 K columns 7.7 -> 5.3 (against tiles through registers, two workgroups per CU).
//
// A lane reads four consecutive columns c0 + 4 (lane / 16) .. + 3 of row lane % 16.  Element s of those four is the
// lane's operand of K step s, for the row block as A operand and as B operand alike (A[i][k] and B[k][j] of the instruction
// both come from lane (k, i) resp. (k, j)), so which column a K slot stands for does not matter.
//
// A mode of at most 8 indices would leave half of the 16 x 16 result unused.  Its tile holds S = 2 (4 for
// n <= 4) ranges of columns stacked in the 16 rows (row s n + i = index i of range s); the diagonal
// n x n sub-blocks of the result are the Gram matrices of the ranges (the rest mixes ranges and is
// dropped), so each instruction covers S times the columns.
#include "asi_gram_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"

#include <cstdio>
#include <cstring>

namespace asi {

constexpr int SG_NT = 512, SG_NW = SG_NT / 64;
constexpr int SG_MAX_WG = 256;             // one workgroup per CU, each walking several tiles
template <int NB> constexpr int sg_row_bytes() { return NB == 1 ? 1024 : 512; }
template <int NB> constexpr int sg_buf_bytes() { return 16 * (NB <= 2 ? NB : 4) * sg_row_bytes<NB>(); }     // 16, 16, 32, 32 KB
template <int NB> constexpr int sg_nbuf() { return NB <= 2 ? 6 : 4; }

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
__global__ __launch_bounds__(SG_NT, 2) void k_subspace_gram(Batch<GramJob> bt) {
    constexpr int RB = sg_row_bytes<NB>(), TC = RB / (int)sizeof(T), BUF = sg_buf_bytes<NB>(), NBUF = sg_nbuf<NB>();
    constexpr int PPR = RB / 16, NP = gram_blocks<NB>();
    constexpr int NL = BUF / 16 / SG_NT;                   // copies per thread and tile
    int lb;
    const GramJob& jb = bt.job[locate(bt, &lb)];
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

// ---- host side ---------------------------------------------------------------------
bool subspace_gram_supported(long long outer, int n, long long inner, int r) {
    if (n < 1 || n > 64 || r < 1 || r > 64 || outer < 1) return false;
    // With four row blocks and one block of ranks the two products of Alg. 1 cost 6 MFMA units per four columns against 10
    // here, and the sums over the waves (80 KB of LDS) are long for the few tiles a workgroup then walks: three 64 x 512 x 7 x 7
    // layers in one launch 29 us here against 14.5 us without LDS (k_subspace_cols), one of 64 x 256 x 14 x 14 14.6 against 10.4.
    if (n > 48 && r <= 16) return false;
    return inner >= 128;                  // a long inner extent: tiles of consecutive columns
}
static int gram_nb(int n) { return (n + 15) / 16; }
static int gram_stack(int n) { return n <= 4 ? 4 : (n <= 8 ? 2 : 1); }
// columns per tile
static int gram_tc(DType xt, int n) { return (n <= 16 ? 1024 * gram_stack(n) : 512) / (xt == F32 ? 4 : 2); }
int subspace_gram_nwg(DType xt, long long outer, int n, long long inner) {
    const long long tc = gram_tc(xt, n), tiles = outer * ((inner + tc - 1) / tc);
    const long long per = (tiles + SG_MAX_WG - 1) / SG_MAX_WG;       // every workgroup walks the same number of tiles
    return (int)((tiles + per - 1) / per);
}

// key: [0] bf16, [1] memory-to-LDS copies, [4..6] NB
bool make_subspace_gram(DType xt, const void* X, long long outer, int n, long long inner, const float* U, int r, double* part,
                        int nwg, int32_t* zero, int nzero, Item* out) {
    if (!subspace_gram_supported(outer, n, inner, r) || !X || !U || !part || nzero < 0 || nzero > 256) return false;
    if (nwg != subspace_gram_nwg(xt, outer, n, inner)) return false;
    GramJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.U = U; jb.part = part; jb.outer = outer; jb.inner = inner; jb.n = n; jb.r = r; jb.nwg = nwg;
    const long long tiles_per_o = (inner + gram_tc(xt, n) - 1) / gram_tc(xt, n), ntiles = outer * tiles_per_o;
    if (ntiles + 8LL * SG_MAX_WG > 0x7fffffffLL) return false;
    jb.tiles_per_o = (int)tiles_per_o; jb.ntiles = (int)ntiles;
    jb.S = gram_stack(n);
    jb.zero = zero; jb.nzero = zero ? nzero : 0;
    const long long esz = xt == F32 ? 4 : 2;
    const bool dma = inner * esz % 16 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0 && n * inner * esz < 0x7fff0000LL;
    const int nb = gram_nb(n);
    *out = Item();
    out->kind = IT_GRAM_MODE;
    out->key = (xt == BF16 ? 1u : 0u) | (dma ? 2u : 0u) | ((unsigned)nb << 4);
    out->nblocks = nwg;
    std::snprintf(out->label, sizeof(out->label), "k_subspace_gram<%s, %d, %s>", xt == F32 ? "float" : "asi::bf16_t", nb,
                  dma ? "true" : "false");
    static_assert(sizeof(GramJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

template <typename T, int NB, bool DMA>
static hipError_t launch_gram_t(dim3 grid, hipStream_t st, const Batch<GramJob>& b) {
    constexpr int ring = sg_nbuf<NB>() * sg_buf_bytes<NB>(), sums = 4 * gram_blocks<NB>() * 256 * 8, lds = ring > sums ? ring : sums;
    static LdsAllowed allowed;
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_subspace_gram<T, NB, DMA>), lds, allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_subspace_gram<T, NB, DMA>), grid, SG_NT, lds, st, b);
    return hipGetLastError();
}
template <typename T, bool DMA>
static hipError_t launch_gram_nb(int nb, dim3 grid, hipStream_t st, const Batch<GramJob>& b) {
    switch (nb) {
        case 1: return launch_gram_t<T, 1, DMA>(grid, st, b);
        case 2: return launch_gram_t<T, 2, DMA>(grid, st, b);
        case 3: return launch_gram_t<T, 3, DMA>(grid, st, b);
        case 4: return launch_gram_t<T, 4, DMA>(grid, st, b);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_gram_items(const Item* const* items, int n, hipStream_t st) {
    Batch<GramJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const unsigned key = items[0]->key;
    const int nb = (int)((key >> 4) & 7u);
    if (key & 1u) return (key & 2u) ? launch_gram_nb<bf16_t, true>(nb, grid, st, b) : launch_gram_nb<bf16_t, false>(nb, grid, st, b);
    return (key & 2u) ? launch_gram_nb<float, true>(nb, grid, st, b) : launch_gram_nb<float, false>(nb, grid, st, b);
}

}  // namespace asi
