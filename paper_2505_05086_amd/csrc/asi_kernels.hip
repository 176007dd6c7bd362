// Generic kernels of the ASI hot path for gfx950 (wave64).
//
// Contractions over a tensor seen from a mode, X[o,i,j] (outer, n, inner):
//   pair: P[i,q]    = sum_{o,j} X[o,i,j] Y[o,q,j]      (A_m V of Alg. 1)
// plus partial-sum reduction and the grouped step 5 of Eq. 14.  Every kernel serves the
// argument blocks of several layers side by side.
#include "asi_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"
#include "asi_zplanes.h"

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

// ---------------------------------------------------------------------------
// pair: P[i,q] = sum_c X[i,c] Y[q,c] on fp64 MFMA.  A workgroup owns 64 rows i x TQ = 16 NBQ outputs q over one split of the
// unfolding columns, in chunks of 64 columns through two LDS buffers (one barrier a chunk); a chunk is requested two before it
// is multiplied and stored one before.  Both tiles lie in LDS with the columns contiguous, pitch 68
// (rows of four banks: 16-byte reads of 16 rows meet every bank once): one 16-byte read gives a lane its operand of four K steps,
// K slot (s, lg) being column 16 b + 4 lg + s on both sides.  Four waves own 16 rows each, the other four take every other block
// of 16 columns on accumulators of their own, added through LDS at the end.
//   A operand (16 i x 4 c) = Xs[16 w + lane % 16][..],  B operand (4 c x 16 q) = Ys[16 nb + lane % 16][..]
// fp32 values are widened to fp64, so every product is exact and the sums are carried in fp64.
// Bound: fp64 MFMA (64 cycles for 16 x 16 x 4) and the vector instructions beside it, which a SIMD issues one after the other:
// per 16 columns and 48 outputs a wave has 12 MFMAs, 4 LDS reads and 16 widenings, and its share of the staging, which ranks up
// to 64 pay once.  Tiles of 64 x 32 outputs (a rank of 40 or 48 then took two of them, and half as many products again in
// padding) with the columns apart in LDS had three reads and three widenings for every two MFMAs: 960 x 40 over 6272 columns 25.0 ->
// 20.6 us, 512 x 48 over 3 x 3136 26.8 -> 20.9, 256 x 32 over 12544 16.4 -> 15.0, 768 x 192 over 2048 21.8 -> 19.4.  A chunk of 64 x 48
// takes 4600 cycles, 3072 of them MFMA; requesting a chunk earlier, two workgroups a CU, or dword copies from memory to LDS
// without registers (22.8) change nothing or lose.
// ---------------------------------------------------------------------------
constexpr int PR_TI = 64, PR_TK = 64, PR_LD = PR_TK + 4, PR_NW = 8, PR_NT = 64 * PR_NW;
typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <int TQ>
constexpr size_t pair_lds() { return 2 * sizeof(float) * PR_LD * (PR_TI + TQ); }

template <typename T> struct Four;                   // four consecutive elements as they lie in memory
template <> struct Four<float> { typedef v4f type; };
template <> struct Four<bf16_t> { typedef uint2 type; };
__device__ __forceinline__ v4f widen4(const v4f& p) { return p; }
__device__ __forceinline__ v4f widen4(const uint2& p) {
    return (v4f){__uint_as_float(p.x << 16), __uint_as_float(p.x & 0xffff0000u), __uint_as_float(p.y << 16), __uint_as_float(p.y & 0xffff0000u)};
}

// one chunk: `left` columns of the split from its first on, tiles in buf
template <int NBQ>
__device__ __forceinline__ void pair_multiply(const float* buf, long long left, int wr, int kgrp, int lg, int ll, v4d (&acc)[NBQ]) {
    const int nkb = (int)((left < PR_TK ? left : PR_TK) + 15) >> 4;
#pragma unroll
    for (int h = 0; h < PR_TK / 32; ++h) {
        const int kb = 2 * h + kgrp;
        if (kb < nkb) {                            // uniform
            const v4f a = *reinterpret_cast<const v4f*>(buf + (16 * wr + ll) * PR_LD + 16 * kb + 4 * lg);
            v4f b[NBQ];
#pragma unroll
            for (int nb = 0; nb < NBQ; ++nb) b[nb] = *reinterpret_cast<const v4f*>(buf + PR_LD * PR_TI + (16 * nb + ll) * PR_LD + 16 * kb + 4 * lg);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const double av = (double)a[u];
#pragma unroll
                for (int nb = 0; nb < NBQ; ++nb) acc[nb] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, (double)b[nb][u], acc[nb], 0, 0, 0);
            }
        }
    }
}
// the K groups add their accumulators through LDS (the tiles are no longer read), then the first stores; out: the split's (n, r)
extern __shared__ __align__(16) float pr_dyn[];
template <int NBQ>
__device__ __forceinline__ void pair_store(double* __restrict__ out, int n, int r, int i0, int q0, int wr, int kgrp, int lg, int ll, const v4d (&acc)[NBQ]) {
    constexpr int TQ = 16 * NBQ;
    double* red = reinterpret_cast<double*>(pr_dyn);              // PR_TI x TQ doubles
    static_assert(pair_lds<TQ>() >= sizeof(double) * PR_TI * TQ, "reduction buffer fits the tiles");
    __syncthreads();
    if (kgrp == 1)
#pragma unroll
        for (int nb = 0; nb < NBQ; ++nb)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[(16 * wr + lg + 4 * v) * TQ + 16 * nb + ll] = acc[nb][v];
    __syncthreads();
    if (kgrp == 0)
#pragma unroll
        for (int nb = 0; nb < NBQ; ++nb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int il = 16 * wr + lg + 4 * v, i = i0 + il, q = q0 + 16 * nb + ll;    // fp64 MFMA result layout
                const double sum = acc[nb][v] + red[il * TQ + 16 * nb + ll];
                if (i < n && q < r) out[(long long)i * r + q] = sum;
            }
}

// FORM: how X (outer, n, inner) lies in memory.  PAIR_LAST: inner = 1, a thread takes four columns of one row.  PAIR_VEC: inner a
// multiple of four and everything aligned, pieces of four columns.  PAIR_ANY: element by element.
// GEN: Y is not read; its tile is the standard-normal V of Alg. 1's first iteration, generated by the thread that stores it.
enum { PAIR_ANY = 0, PAIR_VEC = 1, PAIR_LAST = 2 };
template <typename T, int FORM, bool GEN, int TQ>
__device__ __forceinline__ void pair_tile(const PairJob& jb, int lb) {
    constexpr int TI = PR_TI, NBQ = TQ / 16, BUF = PR_LD * (TI + TQ);
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const float* __restrict__ Y = jb.Y;
    double* __restrict__ part = jb.part;
    const long long outer = jb.outer, inner = jb.inner;
    const int n = jb.n, r = jb.r;
    if (lb >= jb.gx * jb.gy * jb.gz) {             // extra workgroups: another mode's partial-sum tree
        if (threadIdx.x < 256) presum_block(jb.pre.job, jb.pre.njobs, lb - jb.gx * jb.gy * jb.gz);
        return;
    }
    // Neighbouring blocks (one XCD after the renumbering) are the output tiles of the same rows of X,
    // then the row tiles of the same split: the large operand is fetched from memory once.
    lb = xcd_order(lb, jb.gx * jb.gy * jb.gz);
    const int s = lb / (jb.gx * jb.gy), rem = lb - s * (jb.gx * jb.gy), bx = rem / jb.gy, by = rem - bx * jb.gy;
    const long long ncols = outer * inner;
    const int i0 = bx * TI, q0 = by * TQ;
    const long long cbeg = (long long)s * jb.cols_per_split;
    const long long cend = (cbeg + jb.cols_per_split < ncols) ? cbeg + jb.cols_per_split : ncols;
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wave & 3, kgrp = wave >> 2;
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;   // arrival counters of later launches

    // Loads go to addresses that are always valid and what they return stays untouched in registers until stash(): they are one
    // straight run of instructions, all in flight together.  A row or an output past the end reads the last one (its results are
    // dropped); a column past the split's end reads a column inside the tensor and is masked on both sides.  An address is a
    // base that is the same for the wave (scalar unit) plus a lane offset that is worked out once per chunk or per split: the 64-bit
    // arithmetic of a row times inner per load and chunk cost as much as the products.
    constexpr int NXA = TI / 8, NYA = TQ / 8;                // PAIR_ANY: column tid & 63, rows wave + 8 t
    constexpr int NXV = TI / 32, NYV = (TQ + 31) / 32;       // PAIR_VEC: piece tid & 15, rows tid / 16 + 32 t
    constexpr int NXL = TI / 32, NYL = (TQ + 31) / 32;       // PAIR_LAST: (row, group of four columns) e = tid + 512 t
    constexpr int NG = (NBQ + 1) / 2;                        // GEN: (column e & 63, group of four outputs e / 64)
    typedef typename Four<T>::type X4;
    struct Stage {
        T xa[FORM == PAIR_ANY ? NXA : (FORM == PAIR_LAST ? 4 * NXL : 1)];
        X4 xv[FORM == PAIR_VEC ? NXV : 1];
        float ya[GEN ? 4 * NG : (FORM == PAIR_ANY ? NYA : (FORM == PAIR_LAST ? 4 * NYL : 1))];
        v4f yv[!GEN && FORM == PAIR_VEC ? NYV : 1];
    };
    const int cl = FORM == PAIR_VEC ? 4 * (tid & 15) : lane, rl = FORM == PAIR_VEC ? tid >> 4 : wave;
    const long long xplane = (long long)n * inner, yplane = (long long)r * inner;
    // not the last mode: slab and place in it of the chunk to fetch next (uniform)
    long long co = 0, cj = 0;
    if (FORM != PAIR_LAST) { co = cbeg / inner; cj = cbeg - co * inner; }
    const float inv_inner = 1.0f / (float)inner;
    // lane offsets that hold for the whole split
    long long xro[FORM == PAIR_VEC ? NXV : 1], yro[!GEN && FORM == PAIR_VEC ? NYV : 1];
    unsigned xrl = 0, yrl[!GEN && FORM == PAIR_LAST ? NYL : 1];
    if constexpr (FORM == PAIR_VEC) {
#pragma unroll
        for (int t = 0; t < NXV; ++t) { const int i = i0 + rl + 32 * t; xro[t] = (i < n ? i : n - 1) * inner; }
        if constexpr (!GEN)
#pragma unroll
            for (int t = 0; t < NYV; ++t) { const int q = q0 + rl + 32 * t; yro[t] = (q < r ? q : r - 1) * inner; }
    }
    if constexpr (FORM == PAIR_LAST) {
        xrl = (unsigned)(i0 + lane < n ? i0 + lane : n - 1);
        if constexpr (!GEN)
#pragma unroll
            for (int t = 0; t < NYL; ++t) {
                const int q = q0 + (tid + PR_NT * t) % TQ;
                yrl[t] = (unsigned)(q < r ? q : r - 1);
            }
    }
    auto fetch = [&](long long c0, Stage& st) __attribute__((always_inline)) {
        const int lim = (int)(cend - c0 < PR_TK ? cend - c0 : PR_TK);     // columns of the chunk inside the split
        if constexpr (FORM != PAIR_LAST) {
            // this lane's column: slab co + o, place j; a column past the tensor's end reads the chunk's first
            const int in = c0 + cl < ncols ? cl : 0;
            const long long j0 = cj + in;
            const int o = inner < PR_TK ? (int)(((float)(int)j0 + 0.5f) * inv_inner) : (j0 >= inner ? 1 : 0);      // (j0 < 128: exact)
            const long long j = j0 - (inner < PR_TK ? (long long)(o * (int)inner) : (o ? inner : 0));
            const long long xo = o * xplane + j, yo = o * yplane + j;
            const T* __restrict__ xb = X + co * xplane;
            const float* __restrict__ yb = GEN ? nullptr : Y + co * yplane;
            if constexpr (FORM == PAIR_ANY) {
#pragma unroll
                for (int t = 0; t < NXA; ++t) { const int i = i0 + rl + 8 * t; st.xa[t] = (xb + (i < n ? i : n - 1) * inner)[xo]; }
                if constexpr (!GEN)
#pragma unroll
                    for (int t = 0; t < NYA; ++t) { const int q = q0 + rl + 8 * t; st.ya[t] = (yb + (q < r ? q : r - 1) * inner)[yo]; }
            } else {
#pragma unroll
                for (int t = 0; t < NXV; ++t) st.xv[t] = *reinterpret_cast<const X4*>(xb + (xo + xro[t]));
                if constexpr (!GEN)
#pragma unroll
                    for (int t = 0; t < NYV; ++t) st.yv[t] = *reinterpret_cast<const v4f*>(yb + (yo + yro[t]));
            }
            cj += PR_TK;
            if (inner < PR_TK) { const int d = (int)(((float)(int)cj + 0.5f) * inv_inner); co += d; cj -= d * inner; }
            else if (cj >= inner) { ++co; cj -= inner; }
        } else {
            // (64 n and 64 r below 2^30: host check)
            const T* __restrict__ xb = X + c0 * (long long)n;
#pragma unroll
            for (int t = 0; t < NXL; ++t)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int c = 4 * (wave + PR_NW * t) + u;             // uniform
                    st.xa[4 * t + u] = (xb + (c < lim ? c : 0) * (long long)n)[xrl];
                }
            if constexpr (!GEN) {
                const float* __restrict__ yb = Y + c0 * (long long)r;
#pragma unroll
                for (int t = 0; t < NYL; ++t) {
                    const int c = 4 * ((tid + PR_NT * t) / TQ);
#pragma unroll
                    for (int u = 0; u < 4; ++u) st.ya[4 * t + u] = yb[(unsigned)(c + u < lim ? c + u : 0) * (unsigned)r + yrl[t]];
                }
            }
        }
        if constexpr (GEN)
#pragma unroll
            for (int t = 0; t < NG; ++t) {
                const int e = tid + PR_NT * t, c = e & 63, g = e >> 6;
                if (g < 4 * NBQ && q0 + 4 * g < r) gauss4(jb.seed_lo, jb.seed_hi, jb.mode, c0 + c, (uint32_t)(q0 / 4 + g), st.ya + 4 * t);
            }
    };
    // FULL: every column of the chunk belongs to the split
    auto stash_as = [&](auto full, int lim, float* buf, const Stage& st) __attribute__((always_inline)) {
        constexpr bool FULL = decltype(full)::value;
        float* xs = buf;
        float* ys = buf + PR_LD * TI;
        auto mask4 = [&](v4f v, int c) __attribute__((always_inline)) {
            if constexpr (!FULL)
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = c + u < lim ? v[u] : 0.f;
            return v;
        };
        if constexpr (FORM == PAIR_ANY) {
            const bool in = FULL || cl < lim;
#pragma unroll
            for (int t = 0; t < NXA; ++t) xs[(rl + 8 * t) * PR_LD + cl] = in ? to_f32(st.xa[t]) : 0.f;
            if constexpr (!GEN)
#pragma unroll
                for (int t = 0; t < NYA; ++t) ys[(rl + 8 * t) * PR_LD + cl] = in ? st.ya[t] : 0.f;
        } else if constexpr (FORM == PAIR_VEC) {
#pragma unroll
            for (int t = 0; t < NXV; ++t) *reinterpret_cast<v4f*>(xs + (rl + 32 * t) * PR_LD + cl) = mask4(widen4(st.xv[t]), cl);
            if constexpr (!GEN)
#pragma unroll
                for (int t = 0; t < NYV; ++t)
                    if (TQ % 32 == 0 || rl + 32 * t < TQ) *reinterpret_cast<v4f*>(ys + (rl + 32 * t) * PR_LD + cl) = mask4(st.yv[t], cl);
        } else {
#pragma unroll
            for (int t = 0; t < NXL; ++t) {
                const int g = wave + PR_NW * t;
                const v4f v = {to_f32(st.xa[4 * t]), to_f32(st.xa[4 * t + 1]), to_f32(st.xa[4 * t + 2]), to_f32(st.xa[4 * t + 3])};
                *reinterpret_cast<v4f*>(xs + lane * PR_LD + 4 * g) = mask4(v, 4 * g);
            }
            if constexpr (!GEN)
#pragma unroll
                for (int t = 0; t < NYL; ++t) {
                    const int e = tid + PR_NT * t, g = e / TQ, q = e - g * TQ;
                    const v4f v = {st.ya[4 * t], st.ya[4 * t + 1], st.ya[4 * t + 2], st.ya[4 * t + 3]};
                    if (TQ % 32 == 0 || g < PR_TK / 4) *reinterpret_cast<v4f*>(ys + q * PR_LD + 4 * g) = mask4(v, 4 * g);
                }
        }
        if constexpr (GEN)
#pragma unroll
            for (int t = 0; t < NG; ++t) {
                const int e = tid + PR_NT * t, c = e & 63, g = e >> 6;
                if (g < 4 * NBQ)
#pragma unroll
                    for (int u = 0; u < 4; ++u) ys[(4 * g + u) * PR_LD + c] = ((FULL || c < lim) && q0 + 4 * g < r) ? st.ya[4 * t + u] : 0.f;
            }
    };
    auto stash = [&](long long c0, float* buf, const Stage& g) __attribute__((always_inline)) {
        if (cend - c0 >= PR_TK) stash_as(std::true_type{}, PR_TK, buf, g);
        else stash_as(std::false_type{}, (int)(cend - c0), buf, g);
    };

    v4d acc[NBQ];
#pragma unroll
    for (int nb = 0; nb < NBQ; ++nb) acc[nb] = (v4d){0.0, 0.0, 0.0, 0.0};
    // chunk c is multiplied while chunk c + 1 is stored and chunk c + 2 is on its way
    Stage g;
    float* cur = pr_dyn;
    float* nxt = pr_dyn + BUF;
    if (cbeg < cend) {
        fetch(cbeg, g);
        stash(cbeg, cur, g);
        if (cbeg + PR_TK < cend) fetch(cbeg + PR_TK, g);
    }
    for (long long c0 = cbeg; c0 < cend; c0 += PR_TK) {
        __syncthreads();                           // this chunk is stored, and the other buffer has been read
        if (c0 + PR_TK < cend) stash(c0 + PR_TK, nxt, g);
        if (c0 + 2 * PR_TK < cend) fetch(c0 + 2 * PR_TK, g);
        pair_multiply<NBQ>(cur, cend - c0, wr, kgrp, lg, ll, acc);
        float* t = cur; cur = nxt; nxt = t;
    }
    pair_store<NBQ>(part + (long long)s * n * r, n, r, i0, q0, wr, kgrp, lg, ll, acc);
}
template <typename T, bool LAST, bool GEN, int TQ>
__global__ __launch_bounds__(PR_NT, 4) void k_pair(Batch<PairJob> bt) {
    int lb;
    const PairJob& jb = bt.job[locate(bt, &lb)];
    pair_tile<T, LAST ? PAIR_LAST : PAIR_ANY, GEN, TQ>(jb, lb);
}
template <typename T, int TQ>
__global__ __launch_bounds__(PR_NT, 4) void k_pair_vec(Batch<PairJob> bt) {
    int lb;
    const PairJob& jb = bt.job[locate(bt, &lb)];
    pair_tile<T, PAIR_VEC, false, TQ>(jb, lb);
}

// Outputs per workgroup and splits of the columns.  Splits for the least modelled time, in cycles: a CU's workgroups, each 256 NBQ
// cycles of MFMA per 16 columns and 88 + 52 NBQ of staging, reads and widenings; 8000 for what lies before the first and after
// the last product; then the partial sums, written and read once at some 1.6 KB a cycle, a round trip for every 16 (32 up to rank
// 32) that gram0 adds up together, and beyond 32 of them a level of the partial-sum tree (one more launch on the chain).
// Three 512 x 48 layers of 3136 columns: 10 | 13 | 17 | 25 | 32 splits 26.8 | 23.4 | 19.8 | 23.7 | 27.1 us, gram0 25.2 up to 16, then 27.4.
// The second round trip is counted a little shorter for ranks of 33 to 48 along the last mode, whose tiles of 48 tie there with more splits:
// 16 | 26 splits in compress of 14 x 295 x 576 at rank 45 109.1 | 106.1 us, 16 x 202 x 376 at 38 90.0 | 86.1 (three layers 112.3 | 106.8), 64 x 52 x 77 at
// 37 70.0 | 67.3 (73.1 | 70.4); ranks of 49 to 64 gain 1 to 2 us alone and lose 4 in three layers.
static long long pair_cols_per_split(long long ncols, int nsplit) {
    const long long cps = (ncols + nsplit - 1) / nsplit;
    return (cps + 15) / 16 * 16;
}
// The fewest tiles of up to four blocks of outputs, all of them as small as that allows.  Along the last mode as elsewhere: tiles of 64 for three
// blocks cost 1 to 5 us more there (ranks 33 to 48 of modes of 640 to 2048, fp32 and bf16: compress 173.5 against 169.2 us, 105.3 against 101.0;
// two or three tiles of 48, ranks 66 to 144, 264.0 against 271.5, 327.7 against 338.9).  But tiles of 32 where the columns are too few for a
// split (128) and every tile has a CU: the launch is one workgroup's chain, and half as long (512 x 64, 54 columns 9.3 -> 7.8 us, 100 11.6 -> 8.9,
// 128 12.0 -> 9.2; rank 40 8.5 -> 7.7, 10.4 -> 8.9, 11.0 -> 9.0; four layers together 9.7 -> 7.8 and 12.3 -> 9.6).
// And for ranks of 49 to 64 over inner extents that are no multiple of four, whose loads go element by element, where 32 splits of such tiles
// still have a CU each: 124 x 50 over 2 x 3935 columns 20.5 -> 15.0 us, 174 x 58 over 7 x 2206 29.6 -> 20.9, 128 x 64 over 64 x 49 16.8 -> 12.4 (eight
// layers 26.9 -> 24.1; the first in eight 33.4 -> 35.8).  Ranks of 33 to 48 gain 2 to 4 us alone and lose as much in batches.
static int pair_tq(long long ncols, int n, long long inner, int r) {
    const int blocks = (r + 15) / 16, gy = (blocks + 3) / 4;
    const long long narrow = (long long)((n + PR_TI - 1) / PR_TI) * ((blocks + 1) / 2);
    if (blocks > 2 && ncols <= 128 && narrow <= 256) return 32;
    if (blocks == 4 && inner > 1 && inner % 4 != 0 && 32 * narrow <= 256) return 32;
    return 16 * ((blocks + gy - 1) / gy);
}
static int pair_best_splits(long long ncols, int n, long long inner, int r) {
    const int tq = pair_tq(ncols, n, inner, r), lot = r > 32 ? 16 : 32;
    const long long tiles = (long long)((n + PR_TI - 1) / PR_TI) * ((r + tq - 1) / tq);
    const double block = 308.0 * (tq / 16) + 88.0, partial = (double)n * r * (16.0 / 1600.0);
    long long maxs = (ncols + 127) / 128;                     // at least 128 columns per split
    maxs = maxs > 64 ? 64 : (maxs < 1 ? 1 : maxs);
    const double second = inner == 1 && r > 32 && r <= 48 ? 8400.0 : 9600.0;
    int best = 1;
    double best_cost = -1.0;
    for (int ns = 1; ns <= (int)maxs; ns += ns < 16 ? 1 : 2) {
        const long long cps = pair_cols_per_split(ncols, ns);
        if (ns > 1 && cps * (ns - 1) >= ncols) continue;      // the last split would be empty
        const long long per_cu = (tiles * ns + 255) >> 8;
        const double cost = (double)(per_cu * (cps >> 4)) * block + (per_cu > 1 ? 16000.0 : 8000.0) + ns * partial +
                            (ns <= lot ? 4800.0 : (ns <= 2 * lot ? second : 19200.0)) + (ns > 32 ? 10000.0 : 0.0);
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = ns; }
    }
    return best;
}
int pair_splits(long long outer, int n, long long inner, int r, bool coarse) {
    const long long ncols = outer * inner;
    const int fine = pair_best_splits(ncols, n, inner, r);
    if (!coarse) return fine;
    // A count and no model of the tiles above: scratch that holds this many partial sums has always been accepted.  The least rounds x (columns of
    // a split, in chunks, + 128) of 512 workgroups of 64 x 32 (64 along the last mode), 256 columns or more a split.
    const int tq = (inner == 1 && r > 32 && ncols >= 4096) ? 64 : 32;
    const long long tiles = (long long)((n + PR_TI - 1) / PR_TI) * ((r + tq - 1) / tq);
    const int maxs = (int)std::max(1LL, std::min(64LL, (ncols + 255) / 256));
    int best = 1;
    long long best_cost = -1;
    for (int ns = 1; ns <= maxs; ++ns) {
        const long long cps = ((ncols + ns - 1) / ns + PR_TK - 1) / PR_TK * PR_TK;
        if (ns > 1 && cps * (ns - 1) >= ncols) continue;
        const long long cost = (tiles * ns + 511) / 512 * (cps + 128) + (ns > 32 ? 600 : 0);
        if (best_cost < 0 || cost < best_cost) { best = ns; best_cost = cost; }
    }
    // (no split may be empty with 16 columns as the unit either)
    while (best > 1 && pair_cols_per_split(ncols, best) * (best - 1) >= ncols) --best;
    return std::min(best, fine);
}

int presum_blocks(const PresumArgs& a) {
    if (a.njobs <= 0 || a.njobs > 4) return -1;
    long long blocks = 0;
    for (int j = 0; j < a.njobs; ++j) {
        const PresumJob& jb = a.job[j];
        if (!jb.in || !jb.out || jb.cnt <= 0 || jb.nsplit <= 0) return -1;
        if (jb.nchunks != (int)((jb.cnt + 255) / 256) || jb.ngroups != (jb.nsplit + 31) / 32) return -1;
        blocks += (long long)jb.nchunks * jb.ngroups;
    }
    return blocks > 0x3fffffffLL ? -1 : (int)blocks;
}

static bool make_pair_any(DType xt, const void* X, long long outer, int n, long long inner, const float* Y, bool gen,
                          unsigned long long seed, int mode, int r, double* part, int nsplit, int32_t* zero, int nzero,
                          const PresumArgs* pre, Item* out) {
    const long long ncols = outer * inner;
    if (ncols <= 0 || n <= 0 || r <= 0 || nsplit <= 0 || !X || (!Y && !gen) || !part || nzero < 0 || nzero > 256) return false;
    if (inner == 1 && (n >= (1 << 24) || r >= (1 << 24))) return false;      // 32-bit offsets inside a chunk of the last mode
    PairJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.outer = outer; jb.inner = inner; jb.cols_per_split = pair_cols_per_split(ncols, nsplit);
    jb.Y = gen ? nullptr : Y; jb.part = part; jb.n = n; jb.r = r;
    jb.seed_lo = (uint32_t)(seed & 0xffffffffu); jb.seed_hi = (uint32_t)(seed >> 32); jb.mode = mode;
    const int tq = pair_tq(ncols, n, inner, r);
    jb.gx = (n + PR_TI - 1) / PR_TI; jb.gy = (r + tq - 1) / tq; jb.gz = nsplit;
    jb.zero = zero; jb.nzero = zero ? nzero : 0;
    if (pre) {
        jb.pre_blocks = presum_blocks(*pre);
        if (jb.pre_blocks < 0) return false;
        jb.pre = *pre;
    }
    const bool vec = inner % 4 == 0 && reinterpret_cast<uintptr_t>(X) % (xt == F32 ? 16 : 8) == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0;
    // (generating takes an order longer: one form of it is enough)
    const int form = inner == 1 ? PAIR_LAST : (vec && !gen ? PAIR_VEC : PAIR_ANY);
    *out = Item();
    out->kind = IT_PAIR;
    out->key = (xt == BF16 ? 1u : 0u) | ((unsigned)form << 1) | (gen ? 8u : 0u) | ((unsigned)(tq / 16 - 1) << 4);
    const char* tn = xt == F32 ? "float" : "asi::bf16_t";
    if (form == PAIR_VEC) std::snprintf(out->label, sizeof(out->label), "k_pair_vec<%s, %d>", tn, tq);
    else std::snprintf(out->label, sizeof(out->label), "k_pair<%s, %s, %s, %d>", tn, form == PAIR_LAST ? "true" : "false", gen ? "true" : "false", tq);
    out->nblocks = jb.gx * jb.gy * jb.gz + jb.pre_blocks;
    static_assert(sizeof(PairJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

bool make_pair(DType xt, const void* X, long long outer, int n, long long inner, const float* Y, int r, double* part,
               int nsplit, int32_t* zero, int nzero, const PresumArgs* pre, Item* out) {
    return make_pair_any(xt, X, outer, n, inner, Y, false, 0, 0, r, part, nsplit, zero, nzero, pre, out);
}
bool make_pair_gauss(DType xt, const void* X, long long outer, int n, long long inner, unsigned long long seed, int mode,
                     int r, double* part, int nsplit, int32_t* zero, int nzero, const PresumArgs* pre, Item* out) {
    return make_pair_any(xt, X, outer, n, inner, nullptr, true, seed, mode, r, part, nsplit, zero, nzero, pre, out);
}

template <typename T, int FORM, bool GEN, int TQ>
static hipError_t launch_pair_one(const Batch<PairJob>& b, dim3 grid, hipStream_t st) {
    constexpr size_t lds = pair_lds<TQ>();
    void (*fn)(Batch<PairJob>);
    if constexpr (FORM == PAIR_VEC) fn = k_pair_vec<T, TQ>;
    else fn = k_pair<T, FORM == PAIR_LAST, GEN, TQ>;
    if (lds > 64 * 1024) {
        static LdsAllowed allowed;
        const hipError_t e = allow_lds(reinterpret_cast<const void*>(fn), lds, allowed);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(fn, grid, PR_NT, lds, st, b);
    return hipGetLastError();
}
template <typename T, int FORM, bool GEN>
static hipError_t launch_pair_size(int tq, const Batch<PairJob>& b, dim3 grid, hipStream_t st) {
    switch (tq) {
        case 16: return launch_pair_one<T, FORM, GEN, 16>(b, grid, st);
        case 32: return launch_pair_one<T, FORM, GEN, 32>(b, grid, st);
        case 48: return launch_pair_one<T, FORM, GEN, 48>(b, grid, st);
        default: return launch_pair_one<T, FORM, GEN, 64>(b, grid, st);
    }
}
hipError_t launch_pair_items(const Item* const* items, int n, hipStream_t st) {
    Batch<PairJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const unsigned key = items[0]->key;
    const int tq = 16 * (1 + (int)((key >> 4) & 3u));
    switch (key & 15u) {
        case 0: return launch_pair_size<float, PAIR_ANY, false>(tq, b, grid, st);
        case 1: return launch_pair_size<bf16_t, PAIR_ANY, false>(tq, b, grid, st);
        case 2: return launch_pair_size<float, PAIR_VEC, false>(tq, b, grid, st);
        case 3: return launch_pair_size<bf16_t, PAIR_VEC, false>(tq, b, grid, st);
        case 4: return launch_pair_size<float, PAIR_LAST, false>(tq, b, grid, st);
        case 5: return launch_pair_size<bf16_t, PAIR_LAST, false>(tq, b, grid, st);
        case 8: return launch_pair_size<float, PAIR_ANY, true>(tq, b, grid, st);
        case 9: return launch_pair_size<bf16_t, PAIR_ANY, true>(tq, b, grid, st);
        case 12: return launch_pair_size<float, PAIR_LAST, true>(tq, b, grid, st);
        case 13: return launch_pair_size<bf16_t, PAIR_LAST, true>(tq, b, grid, st);
        default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------------------
// sum of split partials
// ---------------------------------------------------------------------------
// VEC: four consecutive elements per thread (count a multiple of four, all pointers 16-byte aligned): a quarter of
// the load instructions and workgroups for the same sums in the same order.
template <typename PT, bool VEC>
__global__ __launch_bounds__(256) void k_sum_partials(Batch<SumJob> bt) {
    int lb;
    const SumJob& jb = bt.job[locate(bt, &lb)];
    const PT* __restrict__ part = static_cast<const PT*>(jb.part);
    const long long count = jb.count;
    constexpr int W = VEC ? 4 : 1;
    typedef PT PV4 __attribute__((ext_vector_type(4)));
    typedef float FV4 __attribute__((ext_vector_type(4)));
    typedef std::conditional_t<VEC, PV4, PT> PV;
    typedef std::conditional_t<VEC, FV4, float> FV;
    const long long e = ((long long)lb * 256 + threadIdx.x) * W;
    if (e >= count) return;
    double s[W];
#pragma unroll
    for (int w = 0; w < W; ++w) s[w] = 0.0;
    constexpr int SU = VEC ? 8 : 16;                         // loads in flight per round (a round is one memory latency)
    for (int sp0 = 0; sp0 < jb.nsplit; sp0 += SU) {
        PV t[SU];
#pragma unroll
        for (int u = 0; u < SU; ++u)
            t[u] = *reinterpret_cast<const PV*>(part + ((sp0 + u < jb.nsplit) ? (long long)(sp0 + u) * count + e : e));
#pragma unroll
        for (int u = 0; u < SU; ++u)
#pragma unroll
            for (int w = 0; w < W; ++w) {
                double tv;
                if constexpr (VEC) tv = (double)t[u][w]; else tv = (double)t[u];
                s[w] += (sp0 + u < jb.nsplit) ? tv : 0.0;
            }
    }
    FV* op = reinterpret_cast<FV*>(jb.out + e);
    FV o;
    if constexpr (VEC) {
#pragma unroll
        for (int w = 0; w < W; ++w) o[w] = (float)s[w];
        if (jb.beta) o += *op;
    } else {
        o = (float)s[0];
        if (jb.beta) o = *op + o;
    }
    *op = o;
}

static bool fill_sum(const void* part, bool f64, int nsplit, long long count, float* out, int beta, Item* it) {
    if (count <= 0 || nsplit <= 0 || !part || !out || (count + 255) / 256 > 0x3fffffffLL) return false;
    SumJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.part = part; jb.out = out; jb.count = count; jb.nsplit = nsplit; jb.beta = beta;
    *it = Item();
    const bool vec = count % 4 == 0 && reinterpret_cast<uintptr_t>(part) % 32 == 0 && reinterpret_cast<uintptr_t>(out) % 16 == 0;
    it->kind = f64 ? IT_SUM_F64 : IT_SUM_F32;
    it->key = vec ? 1u : 0u;
    it->nblocks = (int)(((vec ? count / 4 : count) + 255) / 256);
    std::snprintf(it->label, sizeof(it->label), "k_sum_partials<%s, %s>", f64 ? "double" : "float", vec ? "true" : "false");
    std::memcpy(it->arg, &jb, sizeof(jb));
    return true;
}
bool make_sum_partials(const float* part, int nsplit, long long count, float* out, int beta, Item* it) {
    return fill_sum(part, false, nsplit, count, out, beta, it);
}
bool make_sum_partials_f64(const double* part, int nsplit, long long count, float* out, int beta, Item* it) {
    return fill_sum(part, true, nsplit, count, out, beta, it);
}
hipError_t launch_sum_items(const Item* const* items, int n, hipStream_t st) {
    Batch<SumJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const bool vec = items[0]->key & 1u;
    if (items[0]->kind == IT_SUM_F64) {
        if (vec) hipLaunchKernelGGL((k_sum_partials<double, true>), grid, 256, 0, st, b);
        else hipLaunchKernelGGL((k_sum_partials<double, false>), grid, 256, 0, st, b);
    } else {
        if (vec) hipLaunchKernelGGL((k_sum_partials<float, true>), grid, 256, 0, st, b);
        else hipLaunchKernelGGL((k_sum_partials<float, false>), grid, 256, 0, st, b);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Step 5 of Eq. 14 for grouped convolutions
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_expand_grouped(Batch<ExpandJob> bt) {
    int lb;
    const ExpandJob& jb = bt.job[locate(bt, &lb)];
    const int r2 = jb.r2, taps = jb.taps, cg = jb.cg, og = jb.og;
    const long long total = (long long)jb.cout * cg * taps;
    const long long e = (long long)lb * 256 + threadIdx.x;
    if (e >= total) return;
    const int t = (int)(e % taps);
    const int c = (int)((e / taps) % cg);
    const int o = (int)(e / ((long long)taps * cg));
    const float* tp = jb.T + (long long)o * r2 * taps + t;
    const float* up = jb.U2 + ((long long)(o / og) * cg + c) * r2;
    float acc = 0.f;
    for (int j0 = 0; j0 < r2; j0 += 8) {              // eight terms' loads in flight (clamped addresses), summed in order
        float a[8], b[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int j = j0 + u < r2 ? j0 + u : r2 - 1;
            a[u] = tp[(long long)j * taps];
            b[u] = up[j];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (j0 + u < r2) acc = fmaf(a[u], b[u], acc);
    }
    jb.dW[e] = jb.beta ? jb.dW[e] + acc : acc;
}

bool make_expand_grouped(const float* T, const float* U2, float* dW, int cout, int r2, int taps, int cg, int og,
                         int beta, Item* out) {
    const long long total = (long long)cout * cg * taps;
    if (total <= 0 || !T || !U2 || !dW || (total + 255) / 256 > 0x3fffffffLL) return false;
    ExpandJob jb = {T, U2, dW, cout, r2, taps, cg, og, beta};
    *out = Item();
    out->kind = IT_EXPAND;
    out->nblocks = (int)((total + 255) / 256);
    std::snprintf(out->label, sizeof(out->label), "k_expand_grouped");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}
hipError_t launch_expand_items(const Item* const* items, int n, hipStream_t st) {
    Batch<ExpandJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_expand_grouped, grid, 256, 0, st, b);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// The generated V of Alg. 1's first iteration written out, (ncols, r) row-major: what the generating
// variant of k_pair multiplies by.  One thread per (column, group of four outputs).
// ---------------------------------------------------------------------------
struct GaussJob {
    float* V;
    long long ncols;
    int r, ngroups, mode;
    uint32_t seed_lo, seed_hi;
};
__global__ __launch_bounds__(256) void k_gauss_fill(Batch<GaussJob> bt) {
    int lb;
    const GaussJob& jb = bt.job[locate(bt, &lb)];
    const long long e = (long long)lb * 256 + threadIdx.x;
    if (e >= jb.ncols * jb.ngroups) return;
    const long long c = e / jb.ngroups;
    const int g = (int)(e - c * jb.ngroups);
    float z[4];
    gauss4(jb.seed_lo, jb.seed_hi, jb.mode, c, (uint32_t)g, z);
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (4 * g + k < jb.r) jb.V[c * jb.r + 4 * g + k] = z[k];
}
bool make_gauss_fill(unsigned long long seed, int mode, long long ncols, int r, float* V, Item* out) {
    if (ncols <= 0 || r <= 0 || !V || mode < 0) return false;
    const int ng = (r + 3) / 4;
    const long long blocks = (ncols * ng + 255) / 256;
    if (blocks > 0x3fffffffLL) return false;
    GaussJob jb = {V, ncols, r, ng, mode, (uint32_t)(seed & 0xffffffffu), (uint32_t)(seed >> 32)};
    *out = Item();
    out->kind = IT_GAUSS;
    out->nblocks = (int)blocks;
    std::snprintf(out->label, sizeof(out->label), "k_gauss_fill");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}
hipError_t launch_gauss_items(const Item* const* items, int n, hipStream_t st) {
    Batch<GaussJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_gauss_fill, grid, 256, 0, st, b);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Step 5 of Eq. 14, ungrouped, small core: dW[o, c, t] (+)= sum_j T[o, j, t] U2[c, j], T = sum of the partial tensors
// ---------------------------------------------------------------------------
// The output (cout x C x taps) is the only large tensor of this step; T is a few hundred KB, U2 less.  A workgroup
// owns a few output channels o (their (o, t) pairs are the rows m of a 16 MB-row tile) and 256 input channels:
//   1. its tile of T is summed over the split partial tensors (fp64, in their order, rounded once: what the pass
//      that used to write T out computed; every load of up to 16 partial tensors in flight) into LDS as Ts[m][j];
//   2. wave w multiplies it with U2 of its 64 channels on the fp32 MFMA.  Lane (lg, ll) loads its B operands straight
//      from memory, 16 bytes at a time: U2[c = 64 w + 16 nb + ll][16 kb + 4 lg .. + 3], element s being K step s of
//      block kb; the A operand takes the same K slots from one 16-byte LDS read of row ll.  (Which index a K slot
//      stands for does not matter as long as both operands agree.)
//   3. the results of one output channel and a wave's 64 input channels are contiguous in dW: they go through the
//      wave's own LDS block and out as 16-byte pieces (element by element when the rows of dW are not aligned).
// Before, the sum was a launch of its own and the product ran on the tiled kernel, eight workgroups per tile of T for
// a 512-channel layer, each with its own round trips: 6.6 + 16.3 us for a 512 x 512 x 9 gradient.
struct DwFoldJob {
    const float* Tpart;      // (nsplit, cout, r2, taps)
    const float* U2;         // (C, r2)
    float* dW;               // (cout, C, taps)
    int nsplit, cout, C, r2, taps, beta;
    int co_per;              // output channels per workgroup, at most the CO of the instantiation
    int cblocks;             // blocks of 256 input channels
};

// CO: output channels per workgroup at most (1..3 with nine taps, 16 or 32 with one); NS: partial tensors whose loads are in
// flight together (4 where there are no more: with 16 a batch of 7 x 7 layers, three splits each, issued 96 loads per thread
// for 18 words).  The result tiles take the place of T's, so that five workgroups fit the LDS of a CU; the launch bounds make them
// fit its registers too (135 kept three, with accumulators apart; 96 now), and the 1026 of three 512 x 512 x 9 layers run at once:
// 20.7 -> 19.4 us (products 6 us a SIMD).  B operands requested before T's: 12 registers spilled, 21.0.
// Workgroups per CU that an instantiation's registers are kept to where there are four partial tensors at most: five up to 48 ranks, four
// beyond, one fewer where that many would spill one or two registers (weight gradients of 1280 x 320 at rank 64 40.8 -> 40.1 us, of 1280 x 960
// at rank 48 39.2 -> 38.8, of 256 x 256 x 9 the same; 40.7, 38.5 and the same without bounds).
constexpr int dw_fold_wgs(int rp, int co, int ns) {
    if (ns != 4) return 1;
    return (rp <= 48 ? 5 : 4) - ((co == 2 && rp == 48) || (co == 32 && rp >= 48) ? 1 : 0);
}
template <int TAPS, int RP, int CO, int NS>
__global__ __launch_bounds__(256, dw_fold_wgs(RP, CO, NS)) void k_dw_fold(Batch<DwFoldJob> bt) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    constexpr int MB = (CO * TAPS + 15) / 16;              // 16-row blocks of the tile of T
    static_assert(MB == 1 || MB == 2, "at most 32 rows");
    constexpr int MR = 16 * MB;
    constexpr int RPP = RP + 4;                            // LDS pitch of a row in floats
    constexpr int EPT = (CO * RP * TAPS + 255) / 256;      // elements of the tile per thread, at most
    constexpr int KB = RP / 16;
    constexpr int OSW = CO * TAPS * 64;                    // result tile of a wave
    __shared__ __align__(16) float fold_tile[4 * OSW > MR * RPP ? 4 * OSW : MR * RPP];
    float* Ts = fold_tile;
    int lb;
    const DwFoldJob& jb = bt.job[locate(bt, &lb)];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lg = lane >> 4, ll = lane & 15;
    const int r2 = jb.r2, C = jb.C, nsplit = jb.nsplit;
    const int ob = lb / jb.cblocks, cb = lb - ob * jb.cblocks;
    const int o0 = ob * jb.co_per;
    const int nco = (jb.cout - o0 < jb.co_per) ? jb.cout - o0 : jb.co_per;

    // 1. the tile of T: the nco x r2 x TAPS block at o0, contiguous in every partial tensor
    const long long count = (long long)jb.cout * r2 * TAPS;
    const int E = nco * r2 * TAPS;
    const float* tp = jb.Tpart + (long long)o0 * r2 * TAPS;
    double sum[EPT];
#pragma unroll
    for (int k = 0; k < EPT; ++k) sum[k] = 0.0;
    for (int s0 = 0; s0 < nsplit; s0 += NS) {
        float t[EPT][NS];
#pragma unroll
        for (int k = 0; k < EPT; ++k) {
            const int e = tid + 256 * k;
#pragma unroll
            for (int q = 0; q < NS; ++q) {
                // (addresses valid for every lane, nothing between the loads; what nothing needs is dropped at the sum)
                t[k][q] = tp[(long long)(s0 + q < nsplit ? s0 + q : nsplit - 1) * count + (e < E ? e : 0)];
            }
        }
#pragma unroll
        for (int k = 0; k < EPT; ++k)
#pragma unroll
            for (int q = 0; q < NS; ++q) sum[k] += (s0 + q < nsplit) ? (double)t[k][q] : 0.0;
    }
    // B operands of this lane, requested while the tile goes to LDS
    const int cw = cb * 256 + 64 * wave;                   // first input channel of the wave
    v4f bq[4][KB];
    const bool uvec = r2 % 4 == 0 && reinterpret_cast<uintptr_t>(jb.U2) % 16 == 0;
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        const int c = cw + 16 * nb + ll;
        const float* up = jb.U2 + (long long)(c < C ? c : 0) * r2;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const int j0 = 16 * kb + 4 * lg;
            if (uvec) {
                bq[nb][kb] = *reinterpret_cast<const v4f*>(up + (j0 < r2 ? j0 : 0));
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) bq[nb][kb][i] = up[j0 + i < r2 ? j0 + i : 0];
            }
        }
    }
    for (int e = tid; e < MR * RPP; e += 256) Ts[e] = 0.f;                 // rows past nco * TAPS, columns past r2
    __syncthreads();
#pragma unroll
    for (int k = 0; k < EPT; ++k) {
        const int e = tid + 256 * k;
        if (e < E) {
            const int oj = e / TAPS, t_ = e - oj * TAPS;                   // oj = o * r2 + j
            const int o = oj / r2, j = oj - o * r2;
            Ts[(o * TAPS + t_) * RPP + j] = (float)sum[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
        const bool cin = cw + 16 * nb + ll < C;
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int i = 0; i < 4; ++i) bq[nb][kb][i] = (cin && 16 * kb + 4 * lg + i < r2) ? bq[nb][kb][i] : 0.f;
    }

    // 2. the products
    v4f acc[MB][4];
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) acc[mb][nb] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < KB; ++kb) {
        v4f a[MB];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) a[mb] = *reinterpret_cast<const v4f*>(Ts + (16 * mb + ll) * RPP + 16 * kb + 4 * lg);
#pragma unroll
        for (int s_ = 0; s_ < 4; ++s_)
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int nb = 0; nb < 4; ++nb)
                    acc[mb][nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[mb][s_], bq[nb][kb][s_], acc[mb][nb], 0, 0, 0);
    }

    // 3. acc[mb][nb][e_]: row m = 16 mb + 4 lg + e_ = o * TAPS + t, channel cw + 16 nb + ll
    float* os = fold_tile + wave * OSW;
    __syncthreads();                                       // every wave has read its last operand of T
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int e_ = 0; e_ < 4; ++e_) {
            const int m = 16 * mb + 4 * lg + e_;
            const int o = m / TAPS, t_ = m - o * TAPS;
            if (o < nco) {
#pragma unroll
                for (int nb = 0; nb < 4; ++nb) os[o * (64 * TAPS) + (16 * nb + ll) * TAPS + t_] = acc[mb][nb][e_];
            }
        }
    // (LDS serves a wave's accesses in order: no barrier between its own writes and reads)
    const int nch = C - cw < 64 ? C - cw : 64;                             // channels of this wave that exist (may be <= 0)
    const int nval = nch > 0 ? nch * TAPS : 0;
    const bool vec_ok = reinterpret_cast<uintptr_t>(jb.dW) % 16 == 0 && ((long long)C * TAPS) % 4 == 0;
    for (int o = 0; o < nco; ++o) {
        float* orow = jb.dW + ((long long)(o0 + o) * C + cw) * TAPS;
        const float* src = os + o * (64 * TAPS);
        if (vec_ok) {
#pragma unroll
            for (int k = 0; k < (16 * TAPS + 63) / 64; ++k) {
                const int pc = lane + 64 * k;
                if (4 * pc + 3 < nval) {
                    v4f v = *reinterpret_cast<const v4f*>(src + 4 * pc);
                    v4f* dst = reinterpret_cast<v4f*>(orow + 4 * pc);
                    if (jb.beta) v += *dst;
                    *dst = v;
                } else {
                    for (int i = 4 * pc; i < nval; ++i) orow[i] = jb.beta ? orow[i] + src[i] : src[i];
                }
            }
        } else {
            for (int i = lane; i < nval; i += 64) orow[i] = jb.beta ? orow[i] + src[i] : src[i];
        }
    }
}

bool make_dw_fold(const float* Tpart, int nsplit, const float* U2, float* dW, int cout, int C, int r2, int taps, int beta,
                  Item* out) {
    if (!Tpart || !U2 || !dW || nsplit < 1 || cout <= 0 || C <= 0 || r2 <= 0) return false;
    if ((taps != 1 && taps != 9) || r2 > 64) return false;
    if ((long long)cout * r2 * taps >= (1LL << 31)) return false;
    DwFoldJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.Tpart = Tpart; jb.U2 = U2; jb.dW = dW; jb.nsplit = nsplit; jb.cout = cout; jb.C = C; jb.r2 = r2; jb.taps = taps; jb.beta = beta;
    jb.cblocks = (C + 255) / 256;
    // output channels per workgroup: as many as leave ~128 workgroups (a workgroup's time is round trips, not
    // arithmetic, so fewer workgroups deny the other layers' kernels less of the chip), at most what 32 rows (o, t) hold
    const int comax = 32 / taps;
    int co = (int)(((long long)cout * jb.cblocks) / 128);
    co = co < 1 ? 1 : (co > comax ? comax : co);
    jb.co_per = co;
    const int cot = taps == 9 ? co : (co <= 16 ? 16 : 32);          // the instantiation's bound
    const long long blocks = (long long)((cout + co - 1) / co) * jb.cblocks;
    if (blocks > 0x3fffffffLL) return false;
    const int rp = (r2 + 15) / 16 * 16;
    *out = Item();
    out->kind = IT_DW_FOLD;
    out->key = (taps == 9 ? 1u : 0u) | ((unsigned)(rp / 16) << 4) | ((unsigned)cot << 8) | (nsplit <= 4 ? 1u << 16 : 0u);
    out->nblocks = (int)blocks;
    std::snprintf(out->label, sizeof(out->label), "k_dw_fold<%d, %d, %d>", taps, rp, cot);
    static_assert(sizeof(DwFoldJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

hipError_t launch_dw_fold_items(const Item* const* items, int n, hipStream_t st) {
    Batch<DwFoldJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const unsigned key = items[0]->key;
    const int rp16 = (int)((key >> 4) & 15u), cot = (int)((key >> 8) & 63u), taps = (key & 1u) ? 9 : 1;
    for (int j = 0; j < n; ++j) {                        // the tile of T must fit the instantiation
        DwFoldJob dj;
        std::memcpy(&dj, items[j]->arg, sizeof(dj));
        if (dj.co_per > cot || dj.r2 > 16 * rp16 || dj.taps != taps) return hipErrorInvalidValue;
    }
    const bool few = (key >> 16) & 1u;
#define ASI_DF_CASE(TP, R, CO_)                                                               \
    if (taps == TP && rp16 == R / 16 && cot == CO_) {                                         \
        if (few) hipLaunchKernelGGL((k_dw_fold<TP, R, CO_, 4>), grid, 256, 0, st, b);         \
        else hipLaunchKernelGGL((k_dw_fold<TP, R, CO_, 16>), grid, 256, 0, st, b);            \
        return hipGetLastError();                                                             \
    }
#define ASI_DF_R(TP, CO_) ASI_DF_CASE(TP, 16, CO_) ASI_DF_CASE(TP, 32, CO_) ASI_DF_CASE(TP, 48, CO_) ASI_DF_CASE(TP, 64, CO_)
    ASI_DF_R(9, 1) ASI_DF_R(9, 2) ASI_DF_R(9, 3) ASI_DF_R(1, 16) ASI_DF_R(1, 32)
#undef ASI_DF_R
#undef ASI_DF_CASE
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Steps 2 and 3 of Eq. 14, plane by plane (asi_zplanes.h): planes of up to 16 rows share a workgroup, a wave each
// ---------------------------------------------------------------------------
template <int WB, bool VEC>
__global__ __launch_bounds__(256) void k_z_planes(Batch<ZPlanesJob> bt) {
    int lb;
    const ZPlanesJob& jb = bt.job[locate(bt, &lb)];
    z_planes_block<WB, VEC>(jb, lb);
}

// Any number of planes: one launch element by element takes 6.6 to 8.3 us where the two mode products take 7 + 8 to 9 + 9.5 (1 to 15 planes of 33 x 17
// to 63 x 63), and beside G1 a core of 8 to 15 small planes 6.8 to 8.2 us where G1 and the Kronecker product took 6.5 + 8 to 9.7.
// key: [0..3] blocks of 16 columns, [4] VEC
bool make_z_planes(const float* S, long long planes, int r3, int r4, const float* U3, int H, const float* U4, int W, float* Z,
                   Item* out) {
    if (!S || !U3 || !U4 || !Z || planes <= 0) return false;
    if (H < 1 || W < 1 || H > 64 || W > 64 || r3 < 1 || r4 < 1 || r3 > 32 || r4 > 32) return false;
    const bool vec = r3 % 4 == 0 && r4 % 4 == 0 && W % 4 == 0 && reinterpret_cast<uintptr_t>(U3) % 16 == 0 &&
                     reinterpret_cast<uintptr_t>(U4) % 16 == 0 && reinterpret_cast<uintptr_t>(Z) % 16 == 0;
    if (planes > 0x3fffffffLL) return false;
    ZPlanesJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.S = S; jb.U3 = U3; jb.U4 = U4; jb.Z = Z; jb.planes = planes; jb.H = H; jb.W = W; jb.r3 = r3; jb.r4 = r4;
    jb.hbs = H <= 16 ? 1 : (H <= 32 ? 2 : 4);
    const long long per = 4 / jb.hbs;
    jb.blocks = (int)((planes + per - 1) / per);
    const int wb = (W + 15) / 16;
    *out = Item();
    out->kind = IT_Z_PLANES;
    out->key = (unsigned)wb | (vec ? 16u : 0u);
    out->nblocks = jb.blocks;
    std::snprintf(out->label, sizeof(out->label), vec ? "k_z_planes<%d>" : "k_z_planes<%d, false>", wb);
    static_assert(sizeof(ZPlanesJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

hipError_t launch_z_planes_items(const Item* const* items, int n, hipStream_t st) {
    Batch<ZPlanesJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const unsigned key = items[0]->key;
    const int wb = (int)(key & 15u);
    for (int j = 0; j < n; ++j) {                        // every plane must fit the blocks of the instantiation
        ZPlanesJob zj;
        std::memcpy(&zj, items[j]->arg, sizeof(zj));
        if (zj.H > 64 || zj.W > 16 * wb || zj.r3 > 32 || zj.r4 > 32) return hipErrorInvalidValue;
    }
    switch (key) {
        case 1: hipLaunchKernelGGL((k_z_planes<1, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 2: hipLaunchKernelGGL((k_z_planes<2, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 3: hipLaunchKernelGGL((k_z_planes<3, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 4: hipLaunchKernelGGL((k_z_planes<4, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 17: hipLaunchKernelGGL((k_z_planes<1, true>), grid, 256, 0, st, b); return hipGetLastError();
        case 18: hipLaunchKernelGGL((k_z_planes<2, true>), grid, 256, 0, st, b); return hipGetLastError();
        case 19: hipLaunchKernelGGL((k_z_planes<3, true>), grid, 256, 0, st, b); return hipGetLastError();
        case 20: hipLaunchKernelGGL((k_z_planes<4, true>), grid, 256, 0, st, b); return hipGetLastError();
        default: break;
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// The H and W products of the core projection for large planes: Y[p] = U3^T X[p] U4, one workgroup per plane
// ---------------------------------------------------------------------------
// The mirror image of k_z_planes.  Wave w takes rows h = 16 w .. 16 w + 15 of the plane:
//   T1[h, q]  = sum_w X[h, w] U4[w, q]           A = X (row h = ll, 16-byte loads of four w), B = U4
//   Yw[a, q]  = sum_{h of the wave} U3[h, a] T1[h, q]     A = U3^T (row a = ll), B = T1: register s of the first result
// and the partial Y's of a plane's waves are added through LDS in their order.  A plane of up to 16 rows has one wave, four of them a
// workgroup.  VEC: W is a multiple of four and X aligned.
struct CorePlanesJob {
    const float* X;
    const float* U3;
    const float* U4;
    float* Y;
    long long planes;
    int H, W, r3, r4;
    int hbs;             // waves of a plane: 1, 2 or 4
};

template <int WB, bool VEC>
__global__ __launch_bounds__(256) void k_core_planes(Batch<CorePlanesJob> bt) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    __shared__ float red[4][32][33];
    int lb;
    const CorePlanesJob& jb = bt.job[locate(bt, &lb)];
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), hbs = jb.hbs, hb = wave & (hbs - 1), per = 4 / hbs;
    const int H = jb.H, W = jb.W, r3 = jb.r3, r4 = jb.r4;
    const long long plane0 = (long long)lb * per, plane = plane0 + wave / hbs;
    const float* __restrict__ Xp = jb.X + (plane < jb.planes ? plane : plane0) * H * W;      // (past the end: dropped)
    const int h = 16 * hb + ll;

    // operands: all loads first, from addresses valid for every lane; masked afterwards
    v4f xa[WB];                      // X[h][16 wb + 4 lg .. + 3]
    float u4[WB][2][4];              // U4[16 wb + 4 lg + s][16 qb + ll]
    float u3[2][4];                  // U3[16 hb + 4 lg + s][16 ab + ll]
#pragma unroll
    for (int wb = 0; wb < WB; ++wb) {
        const int w0 = 16 * wb + 4 * lg;
        if (VEC) xa[wb] = *reinterpret_cast<const v4f*>(Xp + ((h < H && w0 < W) ? h * W + w0 : 0));
        else
#pragma unroll
            for (int s_ = 0; s_ < 4; ++s_) xa[wb][s_] = Xp[(h < H && w0 + s_ < W) ? h * W + w0 + s_ : 0];
    }
#pragma unroll
    for (int wb = 0; wb < WB; ++wb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int s_ = 0; s_ < 4; ++s_) {
                const int w = 16 * wb + 4 * lg + s_, q = 16 * qb + ll;
                u4[wb][qb][s_] = jb.U4[(w < W && q < r4) ? w * r4 + q : 0];
            }
#pragma unroll
    for (int ab = 0; ab < 2; ++ab)
#pragma unroll
        for (int s_ = 0; s_ < 4; ++s_) {
            const int hh = 16 * hb + 4 * lg + s_, a = 16 * ab + ll;
            u3[ab][s_] = jb.U3[(hh < H && a < r3) ? hh * r3 + a : 0];
        }
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int wb = 0; wb < WB; ++wb) {
        if (VEC) xa[wb] = (h < H && 16 * wb + 4 * lg < W) ? xa[wb] : zero4;
        else
#pragma unroll
            for (int s_ = 0; s_ < 4; ++s_) xa[wb][s_] = (h < H && 16 * wb + 4 * lg + s_ < W) ? xa[wb][s_] : 0.f;
    }
#pragma unroll
    for (int wb = 0; wb < WB; ++wb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int s_ = 0; s_ < 4; ++s_)
                u4[wb][qb][s_] = (16 * wb + 4 * lg + s_ < W && 16 * qb + ll < r4) ? u4[wb][qb][s_] : 0.f;
#pragma unroll
    for (int ab = 0; ab < 2; ++ab)
#pragma unroll
        for (int s_ = 0; s_ < 4; ++s_) u3[ab][s_] = (16 * hb + 4 * lg + s_ < H && 16 * ab + ll < r3) ? u3[ab][s_] : 0.f;

    // T1: t1[qb][e] = T1[16 hb + 4 lg + e][16 qb + ll]
    v4f t1[2] = {zero4, zero4};
#pragma unroll
    for (int wb = 0; wb < WB; ++wb)
#pragma unroll
        for (int s_ = 0; s_ < 4; ++s_)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
                t1[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[wb][s_], u4[wb][qb][s_], t1[qb], 0, 0, 0);
    // this wave's part of Y: y[ab][qb][e] = Yw[16 ab + 4 lg + e][16 qb + ll]; K slot lg of step s is row 16 hb + 4 lg + s
    v4f y[2][2] = {{zero4, zero4}, {zero4, zero4}};
#pragma unroll
    for (int s_ = 0; s_ < 4; ++s_)
#pragma unroll
        for (int ab = 0; ab < 2; ++ab)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb)
                y[ab][qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(u3[ab][s_], t1[qb][s_], y[ab][qb], 0, 0, 0);
#pragma unroll
    for (int ab = 0; ab < 2; ++ab)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int e = 0; e < 4; ++e) red[wave][16 * ab + 4 * lg + e][16 * qb + ll] = y[ab][qb][e];
    __syncthreads();
    const int sz = r3 * r4;
    float* __restrict__ Yp = jb.Y + plane0 * sz;
    if (hbs == 4) {                                        // uniform
        for (int e = tid; e < sz; e += 256) {
            const int a = e / r4, q = e - a * r4;
            Yp[e] = ((red[0][a][q] + red[1][a][q]) + red[2][a][q]) + red[3][a][q];
        }
        return;
    }
    const int left = (int)(jb.planes - plane0 < per ? jb.planes - plane0 : per);
    for (int e = tid; e < left * sz; e += 256) {
        const int pl = e / sz, a = (e - pl * sz) / r4, q = e - pl * sz - a * r4;
        float v = red[pl * hbs][a][q];
        for (int w = 1; w < hbs; ++w) v += red[pl * hbs + w][a][q];
        Yp[e] = v;
    }
}

bool make_core_planes(const float* X, long long planes, int H, int W, const float* U3, int r3, const float* U4, int r4, float* Y,
                      Item* out) {
    if (!X || !U3 || !U4 || !Y || planes <= 0 || planes > 0x3fffffffLL) return false;
    if (H < 1 || W < 1 || H > 64 || W > 64 || r3 < 1 || r4 < 1 || r3 > 32 || r4 > 32) return false;
    const bool vec = W % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0;
    CorePlanesJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.U3 = U3; jb.U4 = U4; jb.Y = Y; jb.planes = planes; jb.H = H; jb.W = W; jb.r3 = r3; jb.r4 = r4;
    jb.hbs = H <= 16 ? 1 : (H <= 32 ? 2 : 4);
    const long long per = 4 / jb.hbs;
    const int wb = (W + 15) / 16;
    *out = Item();
    out->kind = IT_CORE_PLANES;
    out->key = (unsigned)wb | (vec ? 16u : 0u);
    out->nblocks = (int)((planes + per - 1) / per);
    std::snprintf(out->label, sizeof(out->label), vec ? "k_core_planes<%d>" : "k_core_planes<%d, false>", wb);
    static_assert(sizeof(CorePlanesJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

hipError_t launch_core_planes_items(const Item* const* items, int n, hipStream_t st) {
    Batch<CorePlanesJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    const int wb = (int)(items[0]->key & 15u);
    for (int j = 0; j < n; ++j) {                        // every plane must fit the blocks of the instantiation
        CorePlanesJob cj;
        std::memcpy(&cj, items[j]->arg, sizeof(cj));
        if (cj.H > 64 || cj.W > 16 * wb || cj.r3 > 32 || cj.r4 > 32) return hipErrorInvalidValue;
    }
    switch (items[0]->key) {
        case 1: hipLaunchKernelGGL((k_core_planes<1, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 2: hipLaunchKernelGGL((k_core_planes<2, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 3: hipLaunchKernelGGL((k_core_planes<3, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 4: hipLaunchKernelGGL((k_core_planes<4, false>), grid, 256, 0, st, b); return hipGetLastError();
        case 17: hipLaunchKernelGGL((k_core_planes<1, true>), grid, 256, 0, st, b); return hipGetLastError();
        case 18: hipLaunchKernelGGL((k_core_planes<2, true>), grid, 256, 0, st, b); return hipGetLastError();
        case 19: hipLaunchKernelGGL((k_core_planes<3, true>), grid, 256, 0, st, b); return hipGetLastError();
        case 20: hipLaunchKernelGGL((k_core_planes<4, true>), grid, 256, 0, st, b); return hipGetLastError();
        default: break;
    }
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// one launch for the items of several layers
// ---------------------------------------------------------------------------
// key bits of the mode-product kernels that only bound sizes (see asi_ttm.hip): NBR
static unsigned launch_class(const Item& it) {
    if (it.kind == IT_TTM || it.kind == IT_KSPLIT) return it.key & 0x7e00fu;
    if (it.kind == IT_TTM_DUO) return it.key & 0xfu;
    return it.key;
}
bool same_launch(const Item& a, const Item& b) {
    return a.kind == b.kind && a.aux == b.aux && launch_class(a) == launch_class(b);
}

hipError_t launch_items(const Item* const* items, int n, hipStream_t st, char* label_out) {
    if (n <= 0 || n > kMaxBatch) return hipErrorInvalidValue;
    for (int j = 1; j < n; ++j)
        if (!same_launch(*items[0], *items[j])) return hipErrorInvalidValue;
    if (label_out) std::snprintf(label_out, sizeof(items[0]->label), "%s", items[0]->label);
    switch (items[0]->kind) {
        case IT_TTM: case IT_KSPLIT: return launch_ttm_items(items, n, st, label_out);
        case IT_TTM_DUO: return launch_ttm_duo_items(items, n, st, label_out);
        case IT_TTM_STREAM: return launch_ttm_stream_items(items, n, st);
        case IT_TTM_EXPAND: return launch_ttm_expand_items(items, n, st);
        case IT_PAIR: return launch_pair_items(items, n, st);
        case IT_SUM_F32: case IT_SUM_F64: return launch_sum_items(items, n, st);
        case IT_EXPAND: return launch_expand_items(items, n, st);
        case IT_DW_FOLD: return launch_dw_fold_items(items, n, st);
        case IT_Z_PLANES: return launch_z_planes_items(items, n, st);
        case IT_CORE_PLANES: return launch_core_planes_items(items, n, st);
        case IT_GAUSS: return launch_gauss_items(items, n, st);
        case IT_GRAM_MODE: return launch_gram_items(items, n, st);
        case IT_DIGITS: return launch_digits_items(items, n, st);
        case IT_SMALL: return launch_small_items(items, n, st);
        case IT_TINY: return launch_tiny_items(items, n, st);
        case IT_STEPS: return launch_steps_items(items, n, st);
        case IT_LONG: return launch_long_items(items, n, st);
        case IT_PLANES: return launch_planes_items(items, n, st);
        case IT_SPLIT_BF16: case IT_GEMM_BF16: return launch_bf16_items(items, n, st);
        case IT_PRESUM: case IT_ORTHW_GSUM: case IT_GRAM0: case IT_APPLY: case IT_ORTHW_GRAM: case IT_ORTHW_CHOL: case IT_ORTHW_APPLY:
        case IT_ORTH_BIG: case IT_INIT: return launch_orth_items(items, n, st, label_out);
        case IT_CORR_MFMA: case IT_CORR: return launch_corr_items(items, n, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace asi
