// Subspace steps of bf16 activations on the int8 MFMA, as exact as on the fp64 MFMA.
//
// P = A_m V needs sums that keep directions many decades below the largest, which is why it is carried in fp64.  But a bf16
// value has eight significant bits: scaled by a power of two that puts the tensor's largest value below 2^30, every value down
// to 2^-22 of it is an integer x = d_3 2^24 + d_2 2^16 + d_1 2^8 + d_0 with digits of eight bits (-128 .. 127), and
// v_mfma_i32_16x16x64_i8 sums products of digits without rounding (19 cycles for 16 x 16 x 64 multiply-adds, 1080 on the fp64
// MFMA).  Products of digits whose positions add up to the same power share an int32 accumulator; the few sums of a result are put
// together in fp64, once.  The sums are exact, where fp64 rounds after every four products.
//   k_amax_bf16            largest magnitude of the tensor (the scale), one pass per call
//   k_subspace_gram_digits P = (A_m A_m^T) U_prev for short modes and for long fibres of up to 256: the digits of a tile are both
//                          operands, 4 x 4 digit products a block of G
//   k_pair_digits          P = A_m V along a last mode: V (fp32, from the bf16 MFMA product) is cut into four digits by
//                          k_v_digits, relative to the largest entry of its column in a range of rows; 4 x 4 digit products
// A value below 2^-22 of the largest may have bits below the last digit, a rest: 2e-6 of the values of the layer below, 6e-4 to 1e-2
// behind a GELU.  The thread that cuts it puts the rest on a list of its workgroup, and at the end the products of the listed rests are
// added in fp64, in the order of their places.  From the first tile on whose rests do not fit, a workgroup multiplies its tiles on the fp64 MFMA;
// the Gram matrix of a long mode, which would take longer there than V and P do, gives up instead, and k_subspace_long, which the host
// launches behind it, does the step.  So nothing is left out whatever the values: all entries of G and all products of X are those of
// the fp64 forms, and the sums are rounded less often.
// 64 x 197 x 3072, ranks 32, 64, 192, fp64 forms | digits | digits where every tile has more rests than the list takes, us:
//   batch mode 70 | 50 | 103, token mode 173 | 116 + 3 | 26 + 180, hidden mode 320 | 121 and V's digits (18; 11 with three) | 305,
//   largest magnitude 17, the layer-step 1005 | 763 | 1090.
// Bound: a tile's cutting (300 vector instructions a thread), its products and LDS traffic one after the other,
// 2.4 + 3.6 + 2.8 thousand cycles for 197 rows; the fp64 forms were bound by the fp64 MFMA.
#include "asi_device.h"
#include "asi_kernels.h"
#include "asi_lds.h"

#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned short v2us __attribute__((ext_vector_type(2)));
typedef double v4d __attribute__((ext_vector_type(4)));

constexpr int DG_NT = 512;
constexpr int DG_AMAX = 512;             // workgroups of the largest-magnitude pass = partial maxima

// ---- largest magnitude ----------------------------------------------------------------------
struct AmaxJob {
    const v4u* X;                        // 16-byte pieces
    long long pieces;
    unsigned* out;                       // DG_AMAX bit patterns (of the magnitude, as bf16)
    int32_t* zero;
    int nzero;
};
__device__ __forceinline__ unsigned pk_max(unsigned a, unsigned b) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(v2us, a), __builtin_bit_cast(v2us, b)));
}
__device__ __forceinline__ unsigned block_max(unsigned m, unsigned* red) {      // all threads get it; red: DG_NT / 64 words
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, (unsigned)__shfl_xor((int)m, d));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = red[0];
#pragma unroll
    for (int w = 1; w < DG_NT / 64; ++w) m = max(m, red[w]);
    return m;
}
__global__ __launch_bounds__(DG_NT) void k_amax_bf16(Batch<AmaxJob> bt) {
    __shared__ unsigned red[DG_NT / 64];
    int lb;
    const AmaxJob& jb = bt.job[locate(bt, &lb)];
    if (jb.zero && lb == 0 && (int)threadIdx.x < jb.nzero) jb.zero[threadIdx.x] = 0;
    const v4u* __restrict__ X = jb.X;
    constexpr int U = 8;                 // loads in flight per thread
    unsigned m = 0;
    const long long step = (long long)DG_AMAX * DG_NT;
    for (long long p0 = (long long)lb * DG_NT + threadIdx.x; p0 < jb.pieces; p0 += U * step) {
        v4u t[U];
#pragma unroll
        for (int u = 0; u < U; ++u) t[u] = X[p0 + u * step < jb.pieces ? p0 + u * step : p0];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < 4; ++q) m = pk_max(m, t[u][q] & 0x7fff7fffu);
    }
    m = block_max(max(m & 0xffffu, m >> 16), red);
    if (threadIdx.x == 0) jb.out[lb] = m;
}

// the scale 2^s of a tensor (largest magnitude below 2^30 afterwards) and the smallest bf16 pattern whose last bit is at least 1
struct Scale {
    int s;
    float f;
    unsigned low;
    bool finite;
};
__device__ __forceinline__ Scale tensor_scale(const unsigned* __restrict__ amax, unsigned* red) {
    static_assert(DG_AMAX == DG_NT, "one partial maximum per thread");
    const unsigned a = block_max(amax[threadIdx.x], red);
    const int e = (int)(a >> 7) - 127;
    Scale o;
    o.s = a == 0 || 29 - e > 127 ? 127 : 29 - e;
    o.f = __uint_as_float((unsigned)(o.s + 127) << 23);
    o.low = (unsigned)(134 - o.s) << 7;
    o.finite = a < 0x7f80u;
    return o;
}
// eight bf16 values (memory order) as integers; `small` collects the smallest magnitude less one (zero: the largest number)
__device__ __forceinline__ void to_int8(v4u raw, float f, int (&q)[8], unsigned& small) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        q[2 * d] = (int)(f * __uint_as_float(raw[d] << 16));
        q[2 * d + 1] = (int)(f * __uint_as_float(raw[d] & 0xffff0000u));
        const v2us one = {1, 1};
        const unsigned less = __builtin_bit_cast(unsigned, (v2us)(__builtin_bit_cast(v2us, raw[d] & 0x7fff7fffu) - one));
        small = __builtin_bit_cast(unsigned, __builtin_elementwise_min(__builtin_bit_cast(v2us, small), __builtin_bit_cast(v2us, less)));
    }
}
// the four digits of four integers: byte k of out[d] is digit d of q[k]
__device__ __forceinline__ void digits4(int q0, int q1, int q2, int q3, unsigned (&out)[4]) {
    const unsigned a = ((unsigned)q0 + 0x80808080u) ^ 0x80808080u, b = ((unsigned)q1 + 0x80808080u) ^ 0x80808080u;
    const unsigned c = ((unsigned)q2 + 0x80808080u) ^ 0x80808080u, d = ((unsigned)q3 + 0x80808080u) ^ 0x80808080u;
    const unsigned ab0 = __builtin_amdgcn_perm(b, a, 0x05010400u), ab1 = __builtin_amdgcn_perm(b, a, 0x07030602u);   // a0 b0 a1 b1 | a2 b2 a3 b3
    const unsigned cd0 = __builtin_amdgcn_perm(d, c, 0x05010400u), cd1 = __builtin_amdgcn_perm(d, c, 0x07030602u);
    out[0] = __builtin_amdgcn_perm(cd0, ab0, 0x05040100u);
    out[1] = __builtin_amdgcn_perm(cd0, ab0, 0x07060302u);
    out[2] = __builtin_amdgcn_perm(cd1, ab1, 0x05040100u);
    out[3] = __builtin_amdgcn_perm(cd1, ab1, 0x07060302u);
}
// The values with a rest that a workgroup has met
constexpr int DG_LIST = DG_NT;
constexpr int DG_AHEAD = 16;             // entries whose values are on their way together
constexpr unsigned long long DG_NO_PLACE = ~0ull;
struct RestList {
    int count;
    int full[2];                         // a tile of this parity has brought more than there is room for
    unsigned long long place[DG_LIST];   // tile << 32 | row << 16 | column in the tile
    float rest[DG_LIST];                 // what to_int8 cut off
    __device__ __forceinline__ int tile(int e) const { return (int)(place[e] >> 32); }
    __device__ __forceinline__ int row(int e) const { return (int)(place[e] >> 16) & 0xffff; }
    __device__ __forceinline__ int col(int e) const { return (int)place[e] & 0xffff; }
};
__device__ __forceinline__ bool any_below(unsigned small, unsigned low) {
    const unsigned a = small & 0xffffu, b = small >> 16;
    return min(a, b) + 1u < low;
}
// How many entries there may be after `tiles` tiles of a workgroup.  An entry costs 0.2 to 0.4 us at the end (a read of a column or row, and its
// updates), a tile on the fp64 MFMA 4 to 5 us more than its digits: a dozen entries a tile would pay.  Eight, so that a tensor with
// somewhat more is found out in the first tiles (with twelve, the long mode of a GELU output met 12.5 a tile and was given up after 225 us).
__device__ __forceinline__ int list_room(int tiles) { return min(16 + 8 * tiles, DG_LIST); }
// the values of one piece (eight columns of a row) that have a rest; room: entries that there may be so far, DG_LIST at most
__device__ __forceinline__ void list_rests(RestList& l, int tile, int parity, int room, v4u raw, float f, unsigned low, int row, int col) {
    unsigned has = 0;                    // the values to look at: mostly one, and none in most lanes
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const unsigned b = (k & 1 ? raw[k >> 1] >> 16 : raw[k >> 1]) & 0x7fffu;
        has |= b != 0 && b < low ? 1u << k : 0u;
    }
    while (has) {
        const int k = __builtin_ctz(has);
        has &= has - 1;
        const unsigned w = k < 4 ? (k < 2 ? raw[0] : raw[1]) : (k < 6 ? raw[2] : raw[3]);
        const float t = f * __uint_as_float(k & 1 ? w & 0xffff0000u : w << 16), rest = t - (float)(int)t;
        if (rest == 0.f) continue;
        const int e = atomicAdd(&l.count, 1);
        if (e >= room) {
            if (e < DG_LIST) l.place[e] = DG_NO_PLACE;   // (counted, so it has to hold something: the last in order, and of no tile)
            l.full[parity] = 1;
            return;
        }
        l.place[e] = (unsigned long long)(unsigned)tile << 32 | (unsigned)(row << 16 | (col + k));
        l.rest[e] = rest;
    }
}
// Puts the list in the order of the places, whichever thread came first; returns how many there are of the tiles before `end`
__device__ __forceinline__ int sort_rests(RestList& l, int end) {
    static_assert(DG_LIST <= DG_NT && DG_LIST % 8 == 0, "an entry per thread");
    __syncthreads();
    const int n = l.count < DG_LIST ? l.count : DG_LIST, t = threadIdx.x;        // (every slot below n holds a place)
    const unsigned long long mine = t < n ? l.place[t] : DG_NO_PLACE;
    const float rest = t < n ? l.rest[t] : 0.f;
    int listed = 0, before = 0;
    for (int e0 = 0; e0 < n; e0 += 8) {
        unsigned long long p[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) p[u] = l.place[e0 + u];
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (e0 + u < n) {
                before += p[u] < mine ? 1 : 0;
                listed += (unsigned)(p[u] >> 32) < (unsigned)end ? 1 : 0;
            }
    }
    __syncthreads();
    if (mine != DG_NO_PLACE) { l.place[before] = mine; l.rest[before] = rest; }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(listed);
}
__device__ __forceinline__ v4d mfma_f64(float a, float b, v4d c) { return __builtin_amdgcn_mfma_f64_16x16x4f64((double)a, (double)b, c, 0, 0, 0); }
__device__ __forceinline__ v4i mfma_i8(v4i a, v4i b, v4i c) { return __builtin_amdgcn_mfma_i32_16x16x64_i8(a, b, c, 0, 0, 0); }

extern __shared__ __align__(16) unsigned char dg_dyn[];

// ---- P through the Gram matrix --------------------------------------------------------------
// A workgroup walks tiles of all n rows (16 NB of them) x KK blocks of 64 columns.  LDS holds a tile's digits in operand order:
// 1 KB per (column block, digit, row block), 16 bytes = 16 consecutive columns of one row per lane.  G's blocks on and above the
// diagonal are dealt out: KK = 4 (n <= 64): wave w takes column block w % 4 and half of the blocks; KK = 1 (n <= 256): the blocks go
// to `parts` workgroups, each of which cuts the whole tile into digits, and there to the eight waves.  Seven int32 accumulators a
// block hold |sum| < 2^30 for 2^13 columns of a wave (digit products reach 2^14, four share an accumulator).
// KK = 4: from the first tile whose rests find no room on the list, tiles are multiplied on the fp64 MFMA, as wide values in the place of
// their digits: [four columns][row] 16 bytes.  Its result has row lg + 4 v where the int8 one has 4 lg + v, so A's rows are read in that order.
template <int KK> constexpr int gd_pw() { return KK == 4 ? 5 : 6; }      // blocks per wave, at most
constexpr int GD_G = 7;                  // powers of 256 in a product of two values
constexpr int GD_MAX_COLS = 1 << 13;     // columns per wave
struct GramDigitsJob {
    const void* X;                       // (outer, n, inner) bf16
    const float* U;
    double* part;                        // (slices * parts, n, r)
    const unsigned* amax;
    long long outer, inner;
    int tiles_per_o, ntiles;
    int n, r, slices, parts, per_part;   // blocks of G per part
    int32_t* refused;                    // KK = 1: set by a workgroup that has too many rests for its list
};

template <int KK>
__global__ __launch_bounds__(DG_NT, 2) void k_subspace_gram_digits(Batch<GramDigitsJob> bt) {
    constexpr int GD_PW = gd_pw<KK>(), NBX = KK == 4 ? 4 : 16, TC = 64 * KK, BUF = 4 * KK * NBX * 1024, PPR = TC / 8, NL = 16 * NBX * PPR / DG_NT;
    static_assert(NL == 4, "four pieces of eight values per thread");
    __shared__ unsigned red[DG_NT / 64];
    __shared__ RestList list;
    int lb;
    const GramDigitsJob& jb = bt.job[locate_xcd(bt, &lb)];
    const unsigned short* X = static_cast<const unsigned short*>(jb.X);
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = jb.n, r = jb.r, NB = (n + 15) >> 4;
    const long long inner = jb.inner;
    const int slice = lb / jb.parts, part = lb - slice * jb.parts;
    double* __restrict__ out = jb.part + (long long)lb * n * r;
    const Scale sc = tensor_scale(jb.amax, red);
    if (slice >= jb.slices) {                            // (a partial sum that only the fp64 form has)
        for (int e = tid; e < n * r; e += DG_NT) out[e] = 0.0;
        return;
    }
    if (!sc.finite) {                                    // an infinite or NaN entry: no finite sum to be had
        for (int e = tid; e < n * r; e += DG_NT) out[e] = __builtin_nan("");
        return;
    }
    if (tid == 0) list.count = list.full[0] = list.full[1] = 0;

    // this wave's blocks: p0 .. p0 + np - 1 of the row-wise enumeration of the upper triangle
    const int npairs = NB * (NB + 1) / 2, first = part * jb.per_part;
    const int mine = npairs - first < jb.per_part ? npairs - first : jb.per_part;    // of this workgroup
    const int kk = KK == 4 ? wave & 3 : 0, w = KK == 4 ? wave >> 2 : wave, nw = KK == 4 ? 2 : 8;
    const int per_wave = (mine + nw - 1) / nw;
    const int p0 = w * per_wave, np = p0 >= mine ? 0 : (mine - p0 < per_wave ? mine - p0 : per_wave);
    int bi[GD_PW], bj[GD_PW];
    {
        int i = 0, rem = first + p0;
        while (i < NB && rem >= NB - i) { rem -= NB - i; ++i; }
        int j = i + rem;
#pragma unroll
        for (int p = 0; p < GD_PW; ++p) {
            bi[p] = p < np ? i : 0; bj[p] = p < np ? j : 0;
            if (++j >= NB) { ++i; j = i; }
        }
    }

    // pieces of a tile: (row, eight columns); what lies past the rows or columns arrives as zeros
    constexpr unsigned FAR = 0x80000000u;
    constexpr int RU = DG_NT / PPR;      // rows from one piece of a thread to its next: whole row blocks
    static_assert(RU % 16 == 0, "");
    const int prow = tid / PPR, pcol = 8 * (tid % PPR), k8 = (tid % PPR) & 7;
    const unsigned goff = (unsigned)(2 * (prow * inner + pcol)), gstep = (unsigned)(2 * RU * inner);
    const int dst = (((pcol >> 6) * 4) * NBX + (prow >> 4)) * 1024 + ((k8 >> 1) * 16 + (prow & 15)) * 16 + (k8 & 1) * 8;
    v4u raw[NL];
    auto fetch = [&](int tile) __attribute__((always_inline)) {
        const int o = (unsigned)tile / (unsigned)jb.tiles_per_o;
        const long long j0 = (long long)(tile - o * jb.tiles_per_o) * TC;
        const int vc = (int)(inner - j0 < TC ? inner - j0 : TC);
#if defined(__HIP_DEVICE_COMPILE__)
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned short*>(X + (long long)o * n * inner + j0), 0,
                                                            (int)(2 * (n * inner - j0)), 0x00027000);
#pragma unroll
        for (int u = 0; u < NL; ++u)
            raw[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(pcol < vc && prow + u * RU < n ? goff + u * gstep : FAR), 0, 0);
#endif
    };
    auto store = [&](unsigned char* buf, int tile, int it) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NL; ++u) {
            unsigned small = 0xffffffffu;
            int q[8];
            to_int8(raw[u], sc.f, q, small);
            unsigned a[4], b[4];
            digits4(q[0], q[1], q[2], q[3], a);
            digits4(q[4], q[5], q[6], q[7], b);
#pragma unroll
            for (int d = 0; d < 4; ++d) *reinterpret_cast<v2u*>(buf + dst + (d * NBX + u * (RU / 16)) * 1024) = (v2u){a[d], b[d]};
            if (any_below(small, sc.low)) list_rests(list, tile, it & 1, list_room(it + 1), raw[u], sc.f, sc.low, prow + u * RU, pcol);
        }
    };
    v4i acc[GD_PW][GD_G];
#pragma unroll
    for (int p = 0; p < GD_PW; ++p)
#pragma unroll
        for (int g = 0; g < GD_G; ++g) acc[p][g] = (v4i){0, 0, 0, 0};
    auto operand = [&](const unsigned char* buf, int block, v4i (&d)[4]) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < 4; ++k) d[k] = *reinterpret_cast<const v4i*>(buf + ((kk * 4 + k) * NBX + block) * 1024 + lane * 16);
    };
    auto multiply = [&](const unsigned char* buf) __attribute__((always_inline)) {
        v4i a[4];
#pragma unroll
        for (int p = 0; p < GD_PW; ++p)
            if (p < np) {                                // uniform
                v4i b[4];
                operand(buf, bj[p], b);
                if (p == 0 || bi[p] != bi[p ? p - 1 : 0]) operand(buf, bi[p], a);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[p][i + j] = mfma_i8(a[i], b[j], acc[p][i + j]);
            }
    };

    if (slice < jb.ntiles) fetch(slice);
    __syncthreads();                                     // the list is empty
    if (slice < jb.ntiles) store(dg_dyn, slice, 0);
    if (slice + jb.slices < jb.ntiles) fetch(slice + jb.slices);
    int it = 0, tile = slice;
#pragma unroll 1
    for (; tile < jb.ntiles; tile += jb.slices, ++it) {
        unsigned char* cur = dg_dyn + (it & 1) * BUF;
        __syncthreads();                                 // this tile's digits are there, the other buffer is no longer read
        // (the flag of this parity is written again behind the next barrier only: the same for all waves)
        if (__builtin_amdgcn_readfirstlane(list.full[it & 1])) break;
        int others = 0;                                  // another workgroup has given up: so does this one, behind the next barrier
        if (KK == 1 && tid == 0) others = __hip_atomic_load(jb.refused, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (tile + jb.slices < jb.ntiles) store(dg_dyn + ((it & 1) ^ 1) * BUF, tile + jb.slices, it + 1);
        if (tile + 2 * jb.slices < jb.ntiles) fetch(tile + 2 * jb.slices);
        multiply(cur);
        if (others) list.full[(it & 1) ^ 1] = 1;
    }
    if (KK == 1 && tile < jb.ntiles) {                   // uniform
        if (tid == 0) __hip_atomic_store(jb.refused, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    const int listed = sort_rests(list, tile);
    if (KK == 1 && __builtin_amdgcn_readfirstlane(list.full[it & 1])) return;        // (others, in the last tile)
    // this wave's sums in fp64
    const double unit = ldexp(1.0, -2 * sc.s);
    v4d sum[GD_PW];
#pragma unroll
    for (int p = 0; p < GD_PW; ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            double s = 0.0;
#pragma unroll
            for (int g = GD_G - 1; g >= 0; --g) s = fma(s, 256.0, (double)acc[p][g][v]);
            sum[p][v] = s * unit;
        }
    if constexpr (KK == 4) if (tile < jb.ntiles) {       // uniform
        constexpr int ROWS = 16 * NBX;
        static_assert(4 * ROWS * TC == BUF, "a wide tile takes the place of its digits");
        auto store_wide = [&](unsigned char* buf) __attribute__((always_inline)) {
            // row ^ piece: a wave's pieces of one row would all start at one bank
            v4f* to = reinterpret_cast<v4f*>(buf) + (pcol >> 2) * ROWS + (prow ^ ((pcol >> 3) & 15));
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                float x[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) x[k] = __uint_as_float(k & 1 ? raw[u][k >> 1] & 0xffff0000u : raw[u][k >> 1] << 16);
                to[u * RU] = (v4f){x[0], x[1], x[2], x[3]};
                to[u * RU + ROWS] = (v4f){x[4], x[5], x[6], x[7]};
            }
        };
        const int arow = 4 * (ll & 3) + (ll >> 2);
        // four steps of sixteen columns, of which a lane group has four; the next step's operands are read under the products of this one
        auto multiply_wide = [&](const v4f* w4, auto full) __attribute__((always_inline)) {
            v4f a[2][GD_PW], b[2][GD_PW];
            auto operands = [&](int q) __attribute__((always_inline)) {
#pragma unroll
                for (int p = 0; p < GD_PW; ++p)
                    if (full() || p < np) {              // uniform
                        a[q & 1][p] = w4[4 * q * ROWS + 16 * bi[p] + (arow ^ (8 * kk + 2 * q + (lg >> 1) & 15))];
                        b[q & 1][p] = w4[4 * q * ROWS + 16 * bj[p] + (ll ^ (8 * kk + 2 * q + (lg >> 1) & 15))];
                    }
            };
            operands(0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q < 3) operands(q + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int p = 0; p < GD_PW; ++p)
                        if (full() || p < np) sum[p] = mfma_f64(a[q & 1][p][s], b[q & 1][p][s], sum[p]);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        fetch(tile);
        store_wide(dg_dyn);
        if (tile + jb.slices < jb.ntiles) fetch(tile + jb.slices);
#pragma unroll 1
        for (int k = 0; tile < jb.ntiles; tile += jb.slices, k ^= 1) {
            __syncthreads();
            if (tile + jb.slices < jb.ntiles) store_wide(dg_dyn + (k ^ 1) * BUF);
            if (tile + 2 * jb.slices < jb.ntiles) fetch(tile + 2 * jb.slices);
            const v4f* w4 = reinterpret_cast<const v4f*>(dg_dyn + k * BUF) + (16 * kk + lg) * ROWS;
            if (np == GD_PW) multiply_wide(w4, std::true_type());
            else multiply_wide(w4, std::false_type());
        }
    }
    // G: block p at p GB, element (i, j) of a block at 17 i + j (a block is read along rows and columns: with
    // 16 doubles a row the second cost 22 us for 197 rows)
    constexpr int GB = 16 * 17;
    __syncthreads();
    double* G = reinterpret_cast<double*>(dg_dyn);
#pragma unroll
    for (int round = 0; round < KK; ++round) {           // the column blocks' shares, in their order
        if (kk == round) {
#pragma unroll
            for (int p = 0; p < GD_PW; ++p)
                if (p < np)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        double* d = G + (p0 + p) * GB + (4 * lg + v) * 17 + ll;
                        *d = round == 0 ? sum[p][v] : *d + sum[p][v];
                    }
        }
        __syncthreads();
    }
    // The listed rests R of digits H: row and column i of G gain R_i x_j, the diagonal element R_i (2 x_i - R_i).  Where both values of a
    // product have one, R_i (H_j + R_j) + H_i R_j is what is missing: the lower row meets the upper one without its rest.  DG_AHEAD columns
    // of X on their way
    // (element (lo, hi) of G belongs to thread hi while the entries of rows lo are added, and to thread lo for those of rows hi)
    for (int e0 = 0; e0 < listed; e0 += DG_AHEAD) {
        unsigned short w[DG_AHEAD];
#pragma unroll
        for (int k = 0; k < DG_AHEAD; ++k) {
            const int e = e0 + k < listed ? e0 + k : 0, t = list.tile(e), o = (unsigned)t / (unsigned)jb.tiles_per_o;
            w[k] = X[((long long)o * n + (tid < n ? tid : 0)) * inner + (long long)(t - o * jb.tiles_per_o) * TC + list.col(e)];
        }
#pragma unroll
        for (int below = 0; below < 2; ++below) {
            if (tid < n)
#pragma unroll
                for (int k = 0; k < DG_AHEAD; ++k) {
                    if (e0 + k >= listed) break;         // uniform
                    const int i = __builtin_amdgcn_readfirstlane(list.row(e0 + k));
                    const int lo = below ? tid : i, hi = below ? i : tid, bl = lo >> 4, bh = hi >> 4;
                    const int at = bl * NB - (bl * (bl - 1)) / 2 + bh - bl - first;
                    if (hi < lo || (below && hi == lo) || at < 0 || at >= mine) continue;
                    const float x = sc.f * __uint_as_float((unsigned)w[k] << 16), rest = list.rest[e0 + k];
                    const double add = (double)rest * unit * (tid == i ? 2.0 * (double)x - (double)rest : (double)(below ? x : (float)(int)x));
                    double* g = G + at * GB;
                    const int a = lo & 15, b = hi & 15;
                    g[17 * a + b] += add;
                    if (bl == bh && a != b) g[17 * b + a] += add;        // (a diagonal block is held in full)
                }
            __syncthreads();
        }
    }
    // P = G U, this workgroup's blocks of G: a wave takes a block of 16 outputs, requests all of U for it at once, and walks its
    // share of the row blocks
    const int nqb = (r + 15) >> 4;
    for (int qb = wave % nqb; qb < nqb; qb += DG_NT / 64) {
        const int q = 16 * qb + ll;
        const int sharing = nqb >= 8 ? 1 : (7 - qb) / nqb + 1;         // waves that take this block of outputs
        float u[NBX][4];
#pragma unroll
        for (int kb = 0; kb < NBX; ++kb)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int k = 16 * kb + 4 * s + lg;
                u[kb][s] = jb.U[(k < n && q < r) ? k * r + q : 0];
            }
        for (int ib = nqb >= 8 ? 0 : wave / nqb; ib < NB; ib += sharing) {
            // element (i, k) of G, i in row block ib: from block (ib, kb) or, below the diagonal, from the transpose of (kb, ib); the
            // next block's elements are read under the products of this one
            v4d o = {0.0, 0.0, 0.0, 0.0}, o1 = {0.0, 0.0, 0.0, 0.0};
            auto place = [&](int kb) __attribute__((always_inline)) {
                const int lo = ib < kb ? ib : kb, hi = ib < kb ? kb : ib;
                const int at = lo * NB - (lo * (lo - 1)) / 2 + hi - lo - first;
                return kb < NB && at >= 0 && at < mine ? at : -1;
            };
            auto elements = [&](int kb, int at, double (&x)[4]) __attribute__((always_inline)) {
                const double* g = G + (at < 0 ? 0 : at) * GB + (ib < kb ? 17 * ll + lg : 17 * lg + ll);
                const int step = ib < kb ? 4 : 68;
#pragma unroll
                for (int s = 0; s < 4; ++s) x[s] = g[step * s];
            };
            double x[2][4];
            int at = place(0);
            elements(0, at, x[0]);
#pragma unroll
            for (int kb = 0; kb < NBX; ++kb) {
                const int next = kb + 1 < NBX ? place(kb + 1) : -1;
                if (kb + 1 < NBX) elements(kb + 1, next, x[(kb + 1) & 1]);
                if (at >= 0) {                                         // uniform
#pragma unroll
                    for (int s = 0; s < 4; ++s) {
                        const double uu = 16 * kb + 4 * s + lg < n && q < r ? (double)u[kb][s] : 0.0;
                        if (s & 1) o1 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kb & 1][s], uu, o1, 0, 0, 0);
                        else o = __builtin_amdgcn_mfma_f64_16x16x4f64(x[kb & 1][s], uu, o, 0, 0, 0);
                    }
                }
                at = next;
            }
            o += o1;
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * ib + lg + 4 * v;
                if (i < n && q < r) out[i * r + q] = o[v];
            }
        }
    }
}

// ---- V as digits ------------------------------------------------------------------------------
// V (columns x r, the sum of ks partial products) in four digits relative to the largest entry of an output in a range of columns,
// stored as k_pair_digits copies it to LDS: 1 KB per (chunk of 64 columns, block of 16 outputs, digit), 16 columns per lane.  A
// workgroup per chunk, twice: sums and largest magnitudes, then the digits.  (A workgroup per range and block of outputs that does
// both has 60 workgroups for 12608 x 192 and took 78 us; 8 + 13 so, with three digits.)
// Why four digits: a digit is off by at most half of 2^-29 max |V_q|.  V itself is off by what the two bf16 terms of its factor leave out,
// 2^-18.6 (rms) of the root mean square of a column x_c of X.  Over N columns the digits add 2^-29 max |V_q| |X|_F / sqrt(12) to P_q,
// that adds 2^-18.6 sqrt(sum |x_c|^4 / n); with |V_q| <= |x_c| and |X|_F^2 <= sqrt(N sum |x_c|^4) the first is at most 2^-12.2 sqrt(n) N^(1/4) of
// the second whatever the values, 0.09 for 3072 x 2560 and 0.5 at VD_MAX_N.  (Three digits: up to 256 times as much.)
constexpr int VD_MAX_N = 1 << 16;
struct VDigitsJob {
    const float* V;                      // (ks, ncols, r)
    float* sum;                          // (ncols, r); V itself if there is nothing to add up
    unsigned* most;                      // (chunks, 16 nqb) bit patterns of the largest magnitudes
    unsigned char* out;                  // (nsplit, cps, nqb, 4, 1024)
    double* vscale;                      // (nsplit, 16 nqb): what a unit of an output's digits is worth
    long long ncols;
    int ks, r, nqb, nsplit, cps;         // cps: chunks per split
};
constexpr int VD_NT = 512;
__global__ __launch_bounds__(VD_NT) void k_v_max(Batch<VDigitsJob> bt) {
    __shared__ unsigned most[192];
    int lb;
    const VDigitsJob& jb = bt.job[locate(bt, &lb)];
    const int r = jb.r, tid = threadIdx.x, rp = 16 * jb.nqb;
    const long long c0 = 64LL * lb, all = jb.ncols * r, e0 = c0 * r;
    const int count = (int)(jb.ncols - c0 < 64 ? jb.ncols - c0 : 64) * r;
    if (tid < 192) most[tid] = 0;
    __syncthreads();
    const float inv_r = 1.0f / (float)r;
    constexpr int U = 8;                 // loads in flight; count <= 64 * 192: three rounds at most
    for (int b = tid; b < count; b += U * VD_NT) {
        float v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = jb.V[e0 + (b + u * VD_NT < count ? b + u * VD_NT : b)];
        for (int k = 1; k < jb.ks; ++k) {
            float t[U];
#pragma unroll
            for (int u = 0; u < U; ++u) t[u] = jb.V[k * all + e0 + (b + u * VD_NT < count ? b + u * VD_NT : b)];
#pragma unroll
            for (int u = 0; u < U; ++u) v[u] += t[u];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = b + u * VD_NT;
            if (e >= count) continue;
            if (jb.ks > 1) jb.sum[e0 + e] = v[u];
            const int c = (int)(((float)e + 0.5f) * inv_r);                  // e < 2^14: exact
            atomicMax(&most[e - c * r], __float_as_uint(v[u]) & 0x7fffffffu);            // (Inf and NaN are the largest)
        }
    }
    __syncthreads();
    if (tid < rp) jb.most[(long long)lb * rp + tid] = most[tid];
}
__global__ __launch_bounds__(VD_NT) void k_v_digits(Batch<VDigitsJob> bt) {
    __shared__ int shift[192];           // digits are those of V 2^shift; a number out of reach: not finite
    int lb;
    const VDigitsJob& jb = bt.job[locate(bt, &lb)];
    const int r = jb.r, tid = threadIdx.x, rp = 16 * jb.nqb, z = lb / jb.cps, c_last = 64 * lb;
    const long long left = jb.ncols - c_last;
    const int cols = left < 64 ? (int)left : 64, chunks = (int)((jb.ncols + 63) / 64);
    if (tid < rp) {
        const int k1 = (z + 1) * jb.cps < chunks ? (z + 1) * jb.cps : chunks;
        unsigned m = 0;
#pragma unroll 8
        for (int k = z * jb.cps; k < k1; ++k) m = max(m, jb.most[(long long)k * rp + tid]);
        int e = 0;
        if (m != 0 && m < 0x7f800000u) (void)frexpf(__uint_as_float(m), &e);             // below 2^e
        shift[tid] = m < 0x7f800000u ? 30 - e : 1 << 20;
        if (lb == z * jb.cps) jb.vscale[(long long)z * rp + tid] = m < 0x7f800000u ? ldexp(1.0, e - 30) : __builtin_nan("");
    }
    __syncthreads();
    unsigned char* out = jb.out + (long long)lb * jb.nqb * 4096;
    for (int t = tid; t < 16 * (rp / 4); t += VD_NT) {   // four columns of four outputs
        const int cq = t / (rp / 4), q0 = 4 * (t - cq * (rp / 4));
        float v[4][4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const float* row = jb.sum + (c_last + (4 * cq + c < cols ? 4 * cq + c : 0)) * (long long)r;
            if (r % 4 == 0) {            // uniform: rows of whole 16-byte pieces
                const v4f x = *reinterpret_cast<const v4f*>(row + (q0 < r ? q0 : 0));
#pragma unroll
                for (int q = 0; q < 4; ++q) v[c][q] = x[q];
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q) v[c][q] = row[q0 + q < r ? q0 + q : 0];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) v[c][q] = 4 * cq + c < cols && q0 + q < r ? v[c][q] : 0.f;
        }
        unsigned char* to = out + (q0 >> 4) * 4096 + ((cq >> 2) * 16 + (q0 & 15)) * 16 + 4 * (cq & 3);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int sh = shift[q0 + q];
            int k[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) k[c] = sh < 1 << 20 ? (int)rintf(ldexpf(v[c][q], sh)) : 0;      // (2^30 at most)
            unsigned d[4];
            digits4(k[0], k[1], k[2], k[3], d);
#pragma unroll
            for (int g = 0; g < 4; ++g) *reinterpret_cast<unsigned*>(to + g * 1024 + q * 16) = d[g];
        }
    }
}

// ---- P = A_m V along a last mode ----------------------------------------------------------------
// part[z][i][q] = sum over the columns c of range z of X[c][i] V[c][q]: a workgroup takes 64 rows i and all outputs (up to
// 192), so that X is read and cut once.  Chunks of 64 columns: X through registers (a wave eight columns, a lane one row: bytes of
// consecutive columns are what a lane multiplies, so the cut also transposes), the digits of V copied to LDS as they are.  Two
// buffers each, one barrier a chunk.  Wave w: row blocks 2 (w % 2) and the next, output blocks QB (w / 2) to QB (w / 2) + QB - 1;
// seven int32 accumulators a block.  Chunks from the first one on whose rests find no room on the list are multiplied on the fp64 MFMA, V as
// it is and X wide ([four columns][row] 16 bytes) in the place of their digits.
constexpr int PD_MAX_CPS = 128;          // chunks per range: 4 digit products of 2^14, 64 columns: 2^29
struct PairDigitsJob {
    const void* X;                       // (ncols, n) bf16
    const float* V;                      // (ncols, r)
    const unsigned char* Vd;
    const double* vscale;
    double* part;
    const unsigned* amax;
    long long ncols;
    int n, r, nqb, nsplit, cps, gx;
    int pre_blocks;
    PresumArgs pre;                      // rides along: the first level of the partial-sum tree of other modes
};
template <int QB>
__global__ __launch_bounds__(DG_NT, 2) void k_pair_digits(Batch<PairDigitsJob> bt) {
    constexpr int XB = 4 * 4 * 1024;     // digits of X: [digit][row block]
    __shared__ unsigned red[DG_NT / 64];
    __shared__ RestList list;
    int lb;
    const PairDigitsJob& jb = bt.job[locate(bt, &lb)];
    if (lb >= jb.gx * jb.nsplit) {
        if (threadIdx.x < 256) presum_block(jb.pre.job, jb.pre.njobs, lb - jb.gx * jb.nsplit);
        return;
    }
    lb = xcd_order(lb, jb.gx * jb.nsplit);               // the row tiles of one range share its digits of V
    const unsigned short* X = static_cast<const unsigned short*>(jb.X);
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = jb.n, r = jb.r, nqb = jb.nqb, z = lb / jb.gx, i0 = 64 * (lb - z * jb.gx);
    const long long c_beg = (long long)z * jb.cps * 64, left = jb.ncols - c_beg;
    const int cols = (int)(left < (long long)jb.cps * 64 ? left : (long long)jb.cps * 64), chunks = (cols + 63) >> 6;
    const Scale sc = tensor_scale(jb.amax, red);         // (not finite: neither is V, and its scales are NaN)
    if (tid == 0) list.count = list.full[0] = list.full[1] = 0;
    const int vb = nqb * 4096;                           // bytes of a chunk of V
    unsigned char* const xbuf = dg_dyn;
    unsigned char* const vbuf = dg_dyn + 2 * XB;
    const unsigned char* const vsrc = jb.Vd + (long long)z * jb.cps * vb;

    const int irow = i0 + lane < n ? i0 + lane : n - 1;
    const bool iin = i0 + lane < n;
    const int xdst = (lane >> 4) * 1024 + ((wave >> 1) * 16 + ll) * 16 + (wave & 1) * 8;
    unsigned short raw[8];
    auto fetch = [&](int ch) __attribute__((always_inline)) {
        const int c0 = 64 * ch + 8 * wave;               // scalar
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int c = c0 + k < cols ? c0 + k : cols - 1;
            raw[k] = X[(c_beg + c) * n + irow];
        }
    };
    auto store = [&](int ch, unsigned char* buf) __attribute__((always_inline)) {
        const int c0 = 64 * ch + 8 * wave;
        v4u pk;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const unsigned lo = iin && c0 + 2 * k < cols ? raw[2 * k] : 0u, hi = iin && c0 + 2 * k + 1 < cols ? raw[2 * k + 1] : 0u;
            pk[k] = lo | (hi << 16);
        }
        unsigned small = 0xffffffffu;
        int q[8];
        to_int8(pk, sc.f, q, small);
        unsigned a[4], b[4];
        digits4(q[0], q[1], q[2], q[3], a);
        digits4(q[4], q[5], q[6], q[7], b);
#pragma unroll
        for (int d = 0; d < 4; ++d) *reinterpret_cast<v2u*>(buf + xdst + d * 4096) = (v2u){a[d], b[d]};
        if (any_below(small, sc.low)) list_rests(list, ch, ch & 1, list_room(ch + 1), pk, sc.f, sc.low, lane, 8 * wave);
    };
    auto copy_v = [&](int ch, unsigned char* buf) __attribute__((always_inline)) {
        for (int pc = wave; pc < 4 * nqb; pc += DG_NT / 64) copy16_to_lds(vsrc + (long long)ch * vb, vb, pc * 1024 + lane * 16, buf + pc * 1024);
    };
    constexpr int G = 7;
    v4i acc[2][QB][G];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int k = 0; k < QB; ++k)
#pragma unroll
            for (int g = 0; g < G; ++g) acc[b][k][g] = (v4i){0, 0, 0, 0};
    const int rb = 2 * (wave & 1), qb0 = QB * (wave >> 1);
    auto multiply = [&](const unsigned char* bx, const unsigned char* bv) __attribute__((always_inline)) {
        v4i a[2][4];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int d = 0; d < 4; ++d) a[b][d] = *reinterpret_cast<const v4i*>(bx + d * 4096 + (rb + b) * 1024 + lane * 16);
#pragma unroll
        for (int k = 0; k < QB; ++k)
            if (qb0 + k < nqb) {                         // uniform
                v4i v[4];
#pragma unroll
                for (int d = 0; d < 4; ++d) v[d] = *reinterpret_cast<const v4i*>(bv + ((qb0 + k) * 4 + d) * 1024 + lane * 16);
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
#pragma unroll
                        for (int b = 0; b < 2; ++b) acc[b][k][i + j] = mfma_i8(a[b][i], v[j], acc[b][k][i + j]);
            }
    };
    copy_v(0, vbuf);
    fetch(0);
    __syncthreads();                                     // the list is empty
    store(0, xbuf);
    if (chunks > 1) fetch(1);
    int ch = 0;
#pragma unroll 1
    for (; ch < chunks; ++ch) {
        const int cur = ch & 1;
        wait_copies_and_sync<0>();                       // this chunk's digits are there, the other buffers are no longer read
        // (the flag of this parity is written again behind the next barrier only: the same for all waves)
        if (__builtin_amdgcn_readfirstlane(list.full[cur])) break;
        if (ch + 1 < chunks) {
            copy_v(ch + 1, vbuf + (cur ^ 1) * vb);
            store(ch + 1, xbuf + (cur ^ 1) * XB);
        }
        if (ch + 2 < chunks) fetch(ch + 2);
        multiply(xbuf + cur * XB, vbuf + cur * vb);
    }
    const int listed = sort_rests(list, ch);
    double* __restrict__ out = jb.part + (long long)z * n * r;
    const double unit = ldexp(1.0, -sc.s);
    v4d sum[2][QB];
#pragma unroll
    for (int k = 0; k < QB; ++k) {
        const int q = 16 * (qb0 + k) + ll;
        const double vs = q < r ? jb.vscale[(long long)z * 16 * nqb + q] * unit : 0.0;
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                double s = 0.0;
#pragma unroll
                for (int g = G - 1; g >= 0; --g) s = fma(s, 256.0, (double)acc[b][k][g][v]);
                sum[b][k][v] = s * vs;
            }
    }
    if (ch < chunks) {                                   // uniform
        auto store_wide = [&](int ch, unsigned char* buf) __attribute__((always_inline)) {
            const int c0 = 64 * ch + 8 * wave;
            float x[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k] = iin && c0 + k < cols ? __uint_as_float((unsigned)raw[k] << 16) : 0.f;
            v4f* to = reinterpret_cast<v4f*>(buf) + 2 * wave * 64 + lane;
            to[0] = (v4f){x[0], x[1], x[2], x[3]};
            to[64] = (v4f){x[4], x[5], x[6], x[7]};
        };
        auto copy_wide = [&](int ch, unsigned char* buf) __attribute__((always_inline)) {        // 64 rows of r floats
            const int here = cols - 64 * ch < 64 ? cols - 64 * ch : 64;
            for (int pc = wave; 4 * pc < r; pc += DG_NT / 64)
                copy16_to_lds(jb.V + (c_beg + 64LL * ch) * r, (4 * here * r + 15) & ~15, pc * 1024 + lane * 16, buf + pc * 1024);
        };
        const int arow = 4 * (ll & 3) + (ll >> 2);
        // four steps of sixteen columns, of which a lane group has four; the next step's operands are read under the products of this one
        auto multiply_wide = [&](const v4f* xw, const float* vw, int here, auto full) __attribute__((always_inline)) {
            v4f a[2][2];
            float y[2][QB][4];
            auto operands = [&](int q4) __attribute__((always_inline)) {
                a[q4 & 1][0] = xw[4 * 64 * q4];
                a[q4 & 1][1] = xw[4 * 64 * q4 + 16];
#pragma unroll
                for (int k = 0; k < QB; ++k)
                    if (full() || qb0 + k < nqb)         // uniform
#pragma unroll
                        for (int s = 0; s < 4; ++s) y[q4 & 1][k][s] = vw[(16 * q4 + s) * r + 16 * k];
            };
            operands(0);
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                if (q4 < 3) operands(q4 + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int k = 0; k < QB; ++k)
                        if (full() || qb0 + k < nqb) {
                            const float v = full() || 16 * q4 + s < here ? y[q4 & 1][k][s] : 0.f;        // (what lies behind V's end)
                            sum[0][k] = mfma_f64(a[q4 & 1][0][s], v, sum[0][k]);
                            sum[1][k] = mfma_f64(a[q4 & 1][1][s], v, sum[1][k]);
                        }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        fetch(ch);
        copy_wide(ch, vbuf);
        store_wide(ch, xbuf);
        if (ch + 1 < chunks) fetch(ch + 1);
#pragma unroll 1
        for (int k2 = 0; ch < chunks; ++ch, k2 ^= 1) {
            wait_copies_and_sync<0>();
            if (ch + 1 < chunks) {
                copy_wide(ch + 1, vbuf + (k2 ^ 1) * vb);
                store_wide(ch + 1, xbuf + (k2 ^ 1) * XB);
            }
            if (ch + 2 < chunks) fetch(ch + 2);
            const v4f* xw = reinterpret_cast<const v4f*>(xbuf + k2 * XB) + lg * 64 + 16 * rb + arow;
            const float* vw = reinterpret_cast<const float*>(vbuf + k2 * vb) + 4 * lg * r + 16 * qb0 + ll;
            const int here = cols - 64 * ch;
            if (here >= 64 && qb0 + QB <= nqb) multiply_wide(xw, vw, 64, std::true_type());
            else multiply_wide(xw, vw, here - 4 * lg, std::false_type());
        }
    }
    // the listed rests: row i gains rest V[c]; DG_AHEAD rows of V on their way
    for (int e0 = 0; e0 < listed; e0 += DG_AHEAD) {
        float vv[DG_AHEAD][QB];
#pragma unroll
        for (int e = 0; e < DG_AHEAD; ++e) {
            const int id = e0 + e < listed ? e0 + e : 0;
            const float* row = jb.V + (c_beg + 64LL * list.tile(id) + list.col(id)) * r;
#pragma unroll
            for (int k = 0; k < QB; ++k) vv[e][k] = row[16 * (qb0 + k) + ll < r ? 16 * (qb0 + k) + ll : 0];
        }
#pragma unroll
        for (int e = 0; e < DG_AHEAD; ++e) {
            if (e0 + e >= listed) break;                 // uniform
            const int row = __builtin_amdgcn_readfirstlane(list.row(e0 + e));
            const double rest = ((row >> 2) & 3) == lg ? (double)list.rest[e0 + e] * unit : 0.0;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (row >> 4 == rb + b && (row & 3) == v)            // uniform
#pragma unroll
                        for (int k = 0; k < QB; ++k) sum[b][k][v] = rest != 0.0 ? fma(rest, (double)vv[e][k], sum[b][k][v]) : sum[b][k][v];
        }
    }
#pragma unroll
    for (int k = 0; k < QB; ++k)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = i0 + 16 * (rb + b) + 4 * lg + v, q = 16 * (qb0 + k) + ll;
                if (i < n && q < r) out[(long long)i * r + q] = sum[b][k][v];
            }
}

// ---- host side ----------------------------------------------------------------------------------
bool make_amax_bf16(const void* X, long long numel, unsigned* out_max, int32_t* zero, int nzero, Item* out) {
    if (!X || !out_max || numel < 8 || numel % 8 != 0 || reinterpret_cast<uintptr_t>(X) % 16 != 0 || nzero < 0 || nzero > DG_NT) return false;
    AmaxJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = static_cast<const v4u*>(X); jb.pieces = numel / 8; jb.out = out_max; jb.zero = zero; jb.nzero = zero ? nzero : 0;
    *out = Item();
    out->kind = IT_DIGITS;
    out->key = 0;
    out->nblocks = DG_AMAX;
    std::snprintf(out->label, sizeof(out->label), "k_amax_bf16");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

static bool gram_digits_shape(long long outer, int n, long long inner, GramDigitsJob* jb) {
    if (outer < 1 || n <= 32 || n > 256 || inner < 64 || inner % 8 != 0) return false;
    if (2 * n * inner >= 0x7fff0000LL) return false;             // 32-bit offsets inside a slice of the tensor
    const int nb = (n + 15) / 16, tc = n <= 64 ? 256 : 64, npairs = nb * (nb + 1) / 2;
    const long long tiles_per_o = (inner + tc - 1) / tc, ntiles = outer * tiles_per_o;
    if (ntiles > (1LL << 30)) return false;
    jb->parts = n <= 64 ? 1 : (npairs + 8 * gd_pw<1>() - 1) / (8 * gd_pw<1>());
    jb->per_part = (npairs + jb->parts - 1) / jb->parts;
    const long long most = 256 / jb->parts, per = (ntiles + most - 1) / most;        // one workgroup per CU (LDS)
    if (per * 64 > GD_MAX_COLS) return false;
    jb->slices = (int)((ntiles + per - 1) / per);
    jb->tiles_per_o = (int)tiles_per_o; jb->ntiles = (int)ntiles;
    return true;
}
int subspace_gram_digits_nwg(long long outer, int n, long long inner) {
    GramDigitsJob jb;
    return gram_digits_shape(outer, n, inner, &jb) ? jb.slices * jb.parts : 0;
}
bool make_subspace_gram_digits(const void* X, long long outer, int n, long long inner, const float* U, int r, double* part, int nwg,
                               const unsigned* amax, int32_t* refused, Item* out) {
    GramDigitsJob jb;
    std::memset(&jb, 0, sizeof(jb));
    if (!gram_digits_shape(outer, n, inner, &jb) || jb.slices * jb.parts > nwg || (n > 64 && !refused)) return false;
    if (!X || !U || !part || !amax || r < 1 || reinterpret_cast<uintptr_t>(X) % 16 != 0) return false;
    jb.X = X; jb.U = U; jb.part = part; jb.amax = amax; jb.outer = outer; jb.inner = inner; jb.n = n; jb.r = r; jb.refused = refused;
    *out = Item();
    out->kind = IT_DIGITS;
    out->key = n <= 64 ? 1 : 2;
    out->nblocks = nwg;
    std::snprintf(out->label, sizeof(out->label), "k_subspace_gram_digits<%d>", n <= 64 ? 4 : 1);
    static_assert(sizeof(GramDigitsJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

static int pair_digits_cps(long long ncols, int nsplit) {
    const long long chunks = (ncols + 63) / 64;
    return (int)((chunks + nsplit - 1) / nsplit);
}
int pair_digits_splits(long long ncols, int n, int r) {
    if (ncols < 1024 || ncols >= (1LL << 31) || n < 64 || n > VD_MAX_N || r < 1 || r > 192) return 0;
    const long long gx = (n + 63) / 64, chunks = (ncols + 63) / 64;
    long long ns = gx >= 256 ? 1 : 256 / gx;                     // one workgroup per CU (LDS)
    if (ns > 32) ns = 32;                                        // (a tree level for the partial sums beyond)
    if (ns > chunks / 4) ns = chunks / 4;
    if (ns < 1) ns = 1;
    if (pair_digits_cps(ncols, (int)ns) > PD_MAX_CPS) ns = (chunks + PD_MAX_CPS - 1) / PD_MAX_CPS;
    const int cps = pair_digits_cps(ncols, (int)ns);
    return (int)((chunks + cps - 1) / cps);
}
size_t v_digits_bytes(long long ncols, int r, int nsplit) {
    return (size_t)nsplit * pair_digits_cps(ncols, nsplit) * ((r + 15) / 16) * 4096;
}
size_t v_digits_most(long long ncols, int r) { return (size_t)((ncols + 63) / 64) * 16 * ((r + 15) / 16); }
size_t v_digits_scales(int r, int nsplit) { return (size_t)nsplit * 16 * ((r + 15) / 16); }
bool make_v_digits(const float* V, int ks, float* sum, long long ncols, int r, int nsplit, unsigned* most, unsigned char* digits, double* scales,
                   int step, Item* out) {
    if (!V || !sum || (ks == 1 && sum != V) || !most || !digits || !scales || ks < 1 || nsplit < 1 || r < 1 || r > 192 || ncols >= (1LL << 31)) return false;
    VDigitsJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.V = V; jb.sum = sum; jb.most = most; jb.out = digits; jb.vscale = scales; jb.ncols = ncols; jb.ks = ks; jb.r = r;
    jb.nqb = (r + 15) / 16; jb.nsplit = nsplit; jb.cps = pair_digits_cps(ncols, nsplit);
    *out = Item();
    out->kind = IT_DIGITS;
    out->key = step == 0 ? 7 : 3;
    out->nblocks = (int)((ncols + 63) / 64);
    std::snprintf(out->label, sizeof(out->label), step == 0 ? "k_v_max" : "k_v_digits");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}
bool make_pair_digits(const void* X, long long ncols, int n, const float* V, const unsigned char* digits, const double* scales, int r, double* part,
                      int nsplit, const unsigned* amax, const PresumArgs* pre, Item* out) {
    if (!X || !V || !digits || !scales || !part || !amax || nsplit != pair_digits_splits(ncols, n, r) || nsplit < 1) return false;
    PairDigitsJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.X = X; jb.V = V; jb.Vd = digits; jb.vscale = scales; jb.part = part; jb.amax = amax; jb.ncols = ncols; jb.n = n; jb.r = r;
    jb.nqb = (r + 15) / 16; jb.nsplit = nsplit; jb.cps = pair_digits_cps(ncols, nsplit); jb.gx = (n + 63) / 64;
    if (pre) {
        jb.pre = *pre;
        jb.pre_blocks = presum_blocks(*pre);
        if (jb.pre_blocks < 0) return false;
    }
    const int qb = (jb.nqb + 3) / 4;
    *out = Item();
    out->kind = IT_DIGITS;
    out->key = 3 + qb;                   // 4, 5, 6
    out->nblocks = jb.gx * jb.nsplit + jb.pre_blocks;
    std::snprintf(out->label, sizeof(out->label), "k_pair_digits<%d>", qb);
    static_assert(sizeof(PairDigitsJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

template <int QB>
static hipError_t launch_pair_digits(const Item* const* items, int n, hipStream_t st) {
    Batch<PairDigitsJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    constexpr size_t most = 2 * 16384 + 2 * 4 * QB * 4096;
    static LdsAllowed allowed;
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_pair_digits<QB>), most, allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_pair_digits<QB>, grid, DG_NT, most, st, b);
    return hipGetLastError();
}
template <int KK>
static hipError_t launch_gram_digits(const Item* const* items, int n, hipStream_t st) {
    Batch<GramDigitsJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    constexpr size_t lds = 2 * 65536;
    static LdsAllowed allowed;
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_subspace_gram_digits<KK>), lds, allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_subspace_gram_digits<KK>, grid, DG_NT, lds, st, b);
    return hipGetLastError();
}
hipError_t launch_digits_items(const Item* const* items, int n, hipStream_t st) {
    dim3 grid;
    switch (items[0]->key) {
        case 0: {
            Batch<AmaxJob> b;
            if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
            hipLaunchKernelGGL(k_amax_bf16, grid, DG_NT, 0, st, b);
            return hipGetLastError();
        }
        case 1: return launch_gram_digits<4>(items, n, st);
        case 2: return launch_gram_digits<1>(items, n, st);
        case 3: case 7: {
            Batch<VDigitsJob> b;
            if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
            if (items[0]->key == 7) hipLaunchKernelGGL(k_v_max, grid, VD_NT, 0, st, b);
            else hipLaunchKernelGGL(k_v_digits, grid, VD_NT, 0, st, b);
            return hipGetLastError();
        }
        case 4: return launch_pair_digits<1>(items, n, st);
        case 5: return launch_pair_digits<2>(items, n, st);
        case 6: return launch_pair_digits<3>(items, n, st);
    }
    return hipErrorInvalidValue;
}

}  // namespace asi
