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
#include "asi_subspace_gram.h"

#include <cstdio>
#include <cstring>

namespace asi {

template <typename T, int NB, bool DMA>
__global__ __launch_bounds__(SG_NT, 2) void k_subspace_gram(Batch<GramJob> bt) {
    int lb;
    const GramJob& jb = bt.job[locate(bt, &lb)];
    subspace_gram<T, NB, DMA>(jb, lb);
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
    constexpr int lds = sg_lds_bytes<NB>();
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
