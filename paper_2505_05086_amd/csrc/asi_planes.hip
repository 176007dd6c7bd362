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
#include "asi_subspace_planes.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

template <typename T, int NB, bool DMA>
__global__ __launch_bounds__(PN_NT, NB <= 2 ? 4 : 2) void k_subspace_planes(Batch<PlanesJob> bt) {
    int lb;
    const PlanesJob& jb = bt.job[locate(bt, &lb)];
    subspace_planes<T, NB, DMA>(jb, lb);
}
template <typename T, bool DMA>
__global__ __launch_bounds__(PN_NT, 4) void k_subspace_tiny(Batch<TinyJob> bt) {
    int lb;
    const TinyJob& jb = bt.job[locate(bt, &lb)];
    subspace_tiny<T, DMA>(jb, lb);
}

bool subspace_tiny_supported(int rows, int cols, int r_rows, int r_cols) {
    return rows <= 8 && cols <= 8 && r_rows <= rows && r_cols <= cols;
}
// Planes that a buffer holds (an operand's rows past a plane reach up to 63 elements past the last one: they stay in the buffer).
static int tiny_fit(DType xt, int rows, int cols) { return std::min(512, (TY_BUF - 256) / (rows * cols * (xt == F32 ? 4 : 2)) / 8 * 8); }
// Planes per tile: 128, a workgroup's four waves each a chain of 16 pairs of planes (64 at 512: 10 of a launch's 17 us
// where there are few tiles); twice that and four times while every CU still gets a tile, for fewer partial sums.  Compress, tiles of 512 or as
// many as fit | this: 590 planes of 7 x 1 60.0 -> 51.9 us, 2048 43.6 -> 36.5, 16384 in bf16 60.1 -> 51.6, 65536 83.9 -> 78.2; 2048 of 2 x 2 44.0 -> 35.8,
// 65536 of 4 x 4 84.1 -> 80.9; tiles of 64 take 51.3 and 35.8, but 53.3 for the 16384 and 79.8 for the 65536.
static int tiny_pt(DType xt, long long planes, int rows, int cols) {
    const int fit = tiny_fit(xt, rows, cols);
    int pt = std::min(128, fit);
    while (2 * pt <= fit && planes >= 256LL * 2 * pt) pt *= 2;
    return pt;
}
// two workgroups per CU are resident, and every one walks the same number of tiles
static long long tiny_even(long long tiles) {
    const long long per = (tiles + 511) / 512;
    return (tiles + per - 1) / per;
}
// coarse: no more than one for 128 planes and one for a full buffer
int subspace_tiny_nwg(DType xt, long long planes, int rows, int cols, bool coarse) {
    const long long pt = tiny_pt(xt, planes, rows, cols), fit = tiny_fit(xt, rows, cols), fine = tiny_even((planes + pt - 1) / pt);
    return (int)(coarse ? std::min({fine, tiny_even((planes + 127) / 128), tiny_even((planes + fit - 1) / fit)}) : fine);
}
// key: [0] bf16, [1] memory-to-LDS copies
bool make_subspace_tiny(DType xt, const void* X, long long planes, int rows, int cols, const float* U_rows, int r_rows,
                        double* part_rows, const float* U_cols, int r_cols, double* part_cols, int nwg, Item* out) {
    if (!subspace_tiny_supported(rows, cols, r_rows, r_cols) || !X || !U_rows || !U_cols || !part_rows || !part_cols)
        return false;
    if (planes < 1 || rows < 1 || cols < 1 || nwg < 1 || nwg > subspace_tiny_nwg(xt, planes, rows, cols)) return false;
    TinyJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.planes = planes; jb.pt = tiny_pt(xt, planes, rows, cols); jb.ntiles = (planes + jb.pt - 1) / jb.pt;
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
int subspace_planes_nwg(DType xt, long long planes, int rows, int cols, bool lone) {
    const int pt = planes_pt(xt, planes, rows, cols);
    const long long ntiles = (planes + pt - 1) / pt;
    // Two tiles a workgroup rather than more partial sums than the orthogonalisation adds up without a launch of the summing tree, where these
    // alone would need it.  Compress, a tile a workgroup -> two: 8 x 32 x 16 x 16 20.4 -> 17.6 us, 8 x 32 x 20 x 20 21.5 -> 20.4, 4 x 38 x 28 x 28 28.9 -> 28.4,
    // in bf16 21.3 -> 18.6, 21.4 -> 20.0, 30.6 -> 30.0; beyond 32 x 32 a tile is dearer than the launch (8 x 32 x 40 x 40 31.5 -> 35.8), and where the
    // launch stays, or a pair product carries the tree, nothing is saved (6 x 32 x 28 x 28 22.3 -> 24.7, 3 x 70 x 16 x 16 24.9 -> 25.5).
    if (lone && planes_nb(rows, cols) <= 2 && ntiles > 32 && ntiles <= 64) return (int)((ntiles + 1) / 2);
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
    if (nzero < 0 || nzero > 256 || nwg < 1 || nwg > subspace_planes_nwg(xt, planes, rows, cols, false)) return false;
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
