// Step 4 of Eq. 14 for 3 x 3 taps with a stride of one or two and unit dilation along W, on the bf16 MFMA:
//     T[o,j,kh,kw] = sum_{i,y,x} G1[i,o,y,x] * Zpad[i,j, y*s - p + kh*d, x*t - p + kw]
// The same implicit GEMM as asi_corr.hip (M = o, N = (tap, j), K = (i, y, x); a workgroup owns 64 output channels x 16 core
// channels x 9 taps and walks its share of K in chunks), with every fp32 operand as the exact sum of three bf16 terms
// (x = h + m + l, eight significant bits each, rounded to nearest): a product is the six term products h h, h m, m h, m m, h l,
// l h, each exact in fp32 and summed in fp32; the three left out are below 2^-24 of it, 2^-27.4 (rms) on normal data, where one
// rounding of the sum is up to 2^-24 of the sum so far.  16 x 16 x 32 multiply-adds are 6 x 16 cycles so, 8 x 32 on the fp32 MFMA, and a
// sum of 32 products is rounded once per term product instead of eight times.
//
// A K slot group of a lane is eight consecutive output positions x of one row (rows are padded to a multiple of eight with
// zeros of G1).  Their B operands for the three taps of a kernel row are three windows of ten consecutive entries of a slab
// row: one 16-byte and one 4-byte LDS read per term, the middle window by byte alignment.  With a stride of two the even and the
// odd entries of a slab row are kept apart: the taps 0 and 2 are two windows of the one, tap 1 a window of the other.  Z slabs are cut into terms
// when they are stored to LDS (each serves 64 output channels); G1 goes from memory to the registers of the one wave
// that multiplies it and is cut there, one K block ahead of its products.
//
// Against the fp32 form, us: 256 x 48 x 9 over 8 x 64 x 64 84 -> 49, 128 x 32 x 9 over 16 x 56 x 56 48 -> 35, three of 512 x 48 x 9
// over 16 x 7 x 7 31 -> 21, 960 x 40 x 9 over 24 x 7 x 7 28 -> 18.5, 1024 x 64 x 9 over 32 x 14 x 14 118 -> 78, stride two: 512 x 64 x 9
// over 16 x 14 x 14 44 -> 29; small layers (10 to 15 us, first loads and result) equal or 1 to 2 less.  Bound: a chunk of 256
// positions is 3.3 us of products beside 3 us of vector instructions (200 a K block for the cuts, shifts and copies, 45 a pair of Z),
// which a SIMD issues one after the other.  Error of the weight gradient against 64 bits: 0.905 of the fp32 form's on average over
// 40 layers.
#include "asi_corr.h"
#include "asi_device.h"
#include "asi_lds.h"

#include <cmath>
#include <cstring>
#include <type_traits>

namespace asi {

typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

constexpr int CS_NT = 512;
constexpr int CS_OB = 2, CS_NWO = 2, CS_KG = 4;  // a wave: two blocks of 16 output channels; 2 x 4 waves: channels x K blocks
constexpr int CS_NP = 8;                         // slab pairs per thread and chunk, at most
constexpr int CS_MAX_OCT = 256;                  // groups of eight positions per chunk, at most
constexpr int CS_TS_LD = 16 * 9 + 1;             // result tile: 64 rows of (j, tap)
constexpr size_t CS_LDS_MAX = 160 * 1024;

static size_t split_lds(const CorrPlan& p) {
    const size_t work = 2 * 3 * 2 * (size_t)p.zt + 16 * 4 * (size_t)p.nk, result = sizeof(float) * 2 * CR_TO * CS_TS_LD + 16;
    return work > result ? work : result;
}

// The chunk (ry rows of a map, or ni whole maps) with the fewest cycles for a workgroup's share of K, `want` splits or fewer: a
// round of the eight waves is 2 x 108 products on each SIMD and the vector instructions around them; cutting and storing 512 pairs of
// Z and the barrier come on top (15.8 thousand cycles for a chunk of 256 positions of 64 x 64 maps).
constexpr double CS_ROUND = 5500.0;
static double store_cycles(const CorrGeom& g) { return g.sw == 1 ? 500.0 : 1100.0; }
static bool choose_chunk(const CorrGeom& g, long long want, CorrPlan* p) {
    const long long map = (long long)g.cout * g.Ho * g.Wo;
    double best = 0.0;
    CorrPlan q;
    for (int ni = 1; ni <= g.r1 && ni <= 8; ++ni)
        for (int ry = ni > 1 ? g.Ho : 1; ry <= g.Ho; ++ry) {
            std::memset(&q, 0, sizeof(q));
            q.split = 1;
            q.ni = ni; q.ry = ry;
            q.ow = (g.Wo + 7) / 8;
            q.nyc = (g.Ho + ry - 1) / ry;
            q.rows_in = (ry - 1) * g.sh + 2 * g.dh + 1;
            q.wp = (g.Wo - 1) * g.sw + 3;
            const long long oct = (long long)ni * ry * q.ow, pairs = (long long)ni * 16 * q.rows_in * ((q.wp + 1) / 2);
            if (oct > CS_MAX_OCT || pairs > CS_NP * CS_NT || q.rows_in > 255) break;
            if (4 * ni * map >= (1LL << 30)) break;
            q.nk = (int)(oct + 3) / 4;
            q.px = g.sw * (8 * q.ow + 8);
            q.zj = q.rows_in * q.px;
            if (q.zj / 8 % 2 == 0) q.zj += 8;            // lanes (j) an odd number of 16-byte pieces apart: no two on one bank
            q.zi = 16 * q.zj;
            q.zt = ni * q.zi;
            if (split_lds(q) > CS_LDS_MAX) break;
            q.nchunks = (g.r1 + ni - 1) / ni * q.nyc;
            const long long w = want < q.nchunks ? want : q.nchunks;
            q.cps = (int)((q.nchunks + w - 1) / w);
            q.nsplit = (q.nchunks + q.cps - 1) / q.cps;
            const double cost = q.cps * (CS_ROUND * ((q.nk + CS_KG - 1) / CS_KG) + store_cycles(g) * ((pairs + CS_NT - 1) / CS_NT) + 1000.0);
            if (best == 0.0 || cost < best) { best = cost; *p = q; }
        }
    return best > 0.0;
}

bool corr_split_plan(const CorrGeom& g, CorrPlan* p, bool* cut) {
    *cut = false;
    if (g.kh != 3 || g.kw != 3 || g.sw > 2 || g.dw != 1 || g.Wo > 64) return false;
    if ((long long)g.r1 * g.cout * g.Ho * g.Wo >= (1LL << 31) || (long long)g.r1 * g.r2 * g.H * g.W >= (1LL << 31)) return false;
    // One workgroup per CU (registers) at most, and no more splits than pay: a split takes its share of the walk, and costs the next
    // launch 200 cycles (a round of 16 loads is 1.3 us) and a partial tensor written and read at some 2 TB/s.  Correlation +
    // expansion, splits: 32 x 8 x 9 over 4 x 16 x 16, 16 | 64: 8.7 + 4.0 | 8.5 + 7.2 us; 64 x 16 x 9 over 24 x 7 x 7, 12 | 72: 11.5 + 4.0 |
    // 10.9 + 8.2; 128 x 32 x 9 over 8 x 23 x 23 at stride 2, 22 | 48: 21.4 + 6.2 | 16.0 + 7.3.
    const double rounds = (double)g.r1 * g.Ho * ((g.Wo + 7) / 8) / (4.0 * CS_KG);
    const double stores = (double)g.r1 * g.Ho * g.sh * 16 * (((g.Wo - 1) * g.sw + 4) / 2) / CS_NT;
    const long long even = 1 + (long long)sqrt((1.3 * CS_ROUND * rounds + store_cycles(g) * stores) / (200.0 + 36e-3 * g.cout * g.r2));
    long long want = 256 / corr_plan_tiles(g);
    if (want > even) want = even;
    if (want < 1) want = 1;
    if (!choose_chunk(g, want, p)) return false;
    // A workgroup that would walk a thousand output positions or more of smaller maps is cut in three, as in the fp32 form: more of
    // the sum is then done in fp64, between the splits, and the weight gradient stays as close to 64 bits as it was
    // (512 x 64 x 9 over 16 x 26 x 30: off by 3.3e-7 cut, 4.0e-7 not, 3.8e-7 in the fp32 form; 53 + 17 us uncut).
    *cut = (long long)p->cps * p->ni * p->ry * g.Wo >= 1024 && (long long)g.Ho * g.Wo < 1024;
    return !*cut || choose_chunk(g, 3 * want, p);
}

extern __shared__ __align__(16) unsigned char cs_dyn[];

// two fp32 values as three dwords of two bf16 terms each
__device__ __forceinline__ void split_pair(float a, float b, unsigned& h, unsigned& m, unsigned& l) {
    h = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){a, b}, v2bf));
    const float ra = a - __uint_as_float(h << 16), rb = b - __uint_as_float(h & 0xffff0000u);
    m = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){ra, rb}, v2bf));
    const float sa = ra - __uint_as_float(m << 16), sb = rb - __uint_as_float(m & 0xffff0000u);
    l = __builtin_bit_cast(unsigned, __builtin_convertvector((v2f){sa, sb}, v2bf));
}
// What two fp32 values are, as a dword of two bf16: +-1, 0, +-Inf or NaN.  *huge: one is finite and its first term is not.
__device__ __forceinline__ unsigned sign_or_special(float x, bool* huge) {
    const unsigned u = __float_as_uint(x), e = u & 0x7fffffffu;
    if (e >= 0x7f7f8000u && e < 0x7f800000u) *huge = true;
    return e == 0 ? 0u : (u >> 16 & 0x8000u) | (e < 0x7f800000u ? 0x3f80u : (e == 0x7f800000u ? 0x7f80u : 0x7fc0u));
}
__device__ __forceinline__ unsigned class_pair(float a, float b, bool* huge) { return sign_or_special(a, huge) | sign_or_special(b, huge) << 16; }
// a register's copy (left to itself the compiler reads an operand that starts at an odd register from LDS once more, dword by dword
// and with four lanes to a bank, which costs the LDS as long as the products take)
__device__ __forceinline__ unsigned copy(unsigned x) {
    unsigned y;
    asm("v_mov_b32 %0, %1" : "=v"(y) : "v"(x));
    return y;
}
__device__ __forceinline__ v4f mfma_bf16(v4u a, v4u b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

// RAGGED: output rows are no multiple of eight, the positions past a row's end are cleared.  SW: stride along W
template <int TAPS, bool RAGGED, int SW>
__global__ __launch_bounds__(CS_NT) void k_corr_mfma_split(Batch<CorrJob> bt) {
    static_assert(TAPS == 9, "written for 3 x 3 taps");
    int lb;
    const CorrJob& jb = bt.job[locate_xcd(bt, &lb)];     // the tiles of one split share its G1 rows and Z slabs
    const float* __restrict__ G1 = jb.G1;
    const float* __restrict__ Z = jb.Z;
    const CorrGeom g = jb.g;
    const CorrPlan pl = jb.pl;
    const int bz = lb / (jb.gx * jb.gy), brem = lb - bz * (jb.gx * jb.gy), by = brem / jb.gx, bx = brem - by * jb.gx;
    const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wid = __builtin_amdgcn_readfirstlane(tid >> 6), wo = wid % CS_NWO, kgrp = wid / CS_NWO;
    const int o0 = bx * CR_TO, j0 = by * 16;
    const int HoWo = g.Ho * g.Wo, HW = g.H * g.W;
    const int ch_beg = bz * pl.cps;
    const int ch_end = (ch_beg + pl.cps < pl.nchunks) ? ch_beg + pl.cps : pl.nchunks;
    const int bufsz = 3 * pl.zt;                         // elements of one buffer
    unsigned short* const buf = reinterpret_cast<unsigned short*>(cs_dyn);
    int4* const tab = reinterpret_cast<int4*>(cs_dyn + 4 * (size_t)bufsz);

    // What a thread's loads of Z depend on, whatever the chunk: pair (core channel ii, core channel j, slab row, two columns)
    const int npr = (pl.wp + 1) >> 1, pairs = pl.ni * 16 * pl.rows_in * npr;
    const int nzu = (pairs + CS_NT - 1) / CS_NT;         // uniform
    unsigned off_z[CS_NP];                               // offset inside the chunk's core channels, without the row
    int meta_z[CS_NP];                                   // slab row | ii << 8 | LDS element << 12
    unsigned fix0 = 0, fix1 = 0, step1 = 0;              // the values that lie inside the map's columns; second column's distance
#pragma unroll
    for (int u = 0; u < CS_NP; ++u) {
        off_z[u] = 0; meta_z[u] = 0;
        if (u < nzu) {                                   // uniform
            const int e = u * CS_NT + tid;
            // e < 4096: rounded float quotients are exact
            const int jr = (int)(((float)e + 0.5f) * (1.0f / (float)npr)), m = e - jr * npr;
            const int jj = (int)(((float)jr + 0.5f) * (1.0f / (float)pl.rows_in)), row = jr - jj * pl.rows_in;
            const int ii = jj >> 4, jl = jj & 15, j = j0 + jl;
            const int x0 = 2 * m - g.pw, x1 = x0 + 1;
            const int c0 = min(max(x0, 0), g.W - 1), c1 = min(max(x1, 0), g.W - 1);
            const bool in = e < pairs && j < g.r2;
            fix0 |= (in && x0 == c0) ? (1u << u) : 0u;
            fix1 |= (in && x1 == c1) ? (1u << u) : 0u;
            step1 |= c1 != c0 ? (1u << u) : 0u;
            off_z[u] = e < pairs ? (unsigned)((ii * g.r2 + min(j, g.r2 - 1)) * HW + c0) : 0u;
            meta_z[u] = e < pairs ? row | (ii << 8) | ((ii * pl.zi + jl * pl.zj + row * pl.px + (SW == 1 ? 2 * m : m)) << 12) : -1;
        }
    }
    float z0[CS_NP], z1[CS_NP];
    unsigned zrow = 0;                                   // the fetched pairs whose row lies in the map
    auto fetch_z = [&](int i0, int yc) __attribute__((always_inline)) {
        const int ylo = yc * pl.ry * g.sh - g.ph;
        const float* __restrict__ Zi = Z + (unsigned)(i0 * g.r2) * (unsigned)HW;             // uniform
        zrow = 0;
#pragma unroll
        for (int u = 0; u < CS_NP; ++u)
            if (u < nzu) {                               // uniform
                const int row = ylo + (meta_z[u] & 0xff), rowc = min(max(row, 0), g.H - 1);
                const bool iin = i0 + ((meta_z[u] >> 8) & 15) < g.r1;
                const unsigned off = iin ? off_z[u] + (unsigned)(rowc * g.W) : 0u;
                z0[u] = Zi[off];
                z1[u] = Zi[off + ((step1 >> u) & 1u)];
                zrow |= (row == rowc && iin) ? (1u << u) : 0u;
            }
    };
    bool huge = false, z_special = false;                // what the second walk has met
    auto store_z = [&](unsigned short* b, auto plain) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < CS_NP; ++u)
            if (u < nzu && meta_z[u] >= 0) {
                const float x0 = ((zrow & fix0) >> u) & 1u ? z0[u] : 0.f, x1 = ((zrow & fix1) >> u) & 1u ? z1[u] : 0.f;
                unsigned h, m = 0, l = 0;
                if constexpr (plain()) {
                    h = class_pair(x0, x1, &huge);
                    z_special = z_special || !(fabsf(x0) < INFINITY) || !(fabsf(x1) < INFINITY);
                } else {
                    split_pair(x0, x1, h, m, l);
                }
                unsigned short* d = b + (meta_z[u] >> 12);
                if constexpr (SW == 1) {
                    *reinterpret_cast<unsigned*>(d) = h;
                    *reinterpret_cast<unsigned*>(d + pl.zt) = m;
                    *reinterpret_cast<unsigned*>(d + 2 * pl.zt) = l;
                } else {                                 // an even and an odd entry
                    const int odd = pl.px >> 1;
                    d[0] = (unsigned short)h; d[odd] = (unsigned short)(h >> 16);
                    d[pl.zt] = (unsigned short)m; d[pl.zt + odd] = (unsigned short)(m >> 16);
                    d[2 * pl.zt] = (unsigned short)l; d[2 * pl.zt + odd] = (unsigned short)(l >> 16);
                }
            }
    };

    // G1 of a K block: eight positions of two channels per lane.  Groups past the chunk's rows lie beyond the descriptor's
    // extent and arrive as zeros.
    unsigned arow[CS_OB];
#pragma unroll
    for (int ob = 0; ob < CS_OB; ++ob) {
        const int o = o0 + 16 * (CS_OB * wo + ob) + ll;
        arow[ob] = 4u * (unsigned)((o < g.cout ? o : g.cout - 1) * HoWo);
    }
    v4u araw[CS_OB][2];
    int a_org = 0, a_left = 0;
    auto fetch_a = [&](int i0, int yc, int kb) __attribute__((always_inline)) {
        const int y0 = yc * pl.ry, rows = min(pl.ry, g.Ho - y0), nis = min(pl.ni, g.r1 - i0);
        const int4 t = tab[4 * kb + lg];
        const long long base = (long long)i0 * g.cout * HoWo + (long long)y0 * g.Wo;             // uniform
        const long long left = 4 * ((long long)g.r1 * g.cout * HoWo - base);
        const bool in = (t.z & 0xffff) < rows && (t.z >> 16) < nis;
        const unsigned off = in ? (unsigned)t.y : 0x80000000u;
        a_org = t.x; a_left = t.w;
#if defined(__HIP_DEVICE_COMPILE__)
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(G1 + base), 0, (int)(left < 0x7fffffff ? left : 0x7fffffff), 0x00027000);
#pragma unroll
        for (int ob = 0; ob < CS_OB; ++ob) {
            araw[ob][0] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + arow[ob]), 0, 0);
            araw[ob][1] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + arow[ob] + 16u), 0, 0);
        }
#endif
    };

    v4f acc[CS_OB][9];
    float* Ts = reinterpret_cast<float*>(cs_dyn);
    constexpr int TS_SZ = CR_TO * CS_TS_LD;
    volatile int* const met = reinterpret_cast<int*>(Ts + 2 * TS_SZ);    // behind the tiles: what any thread has met
    // This workgroup's share of K, summed into the tiles Ts.  plain: of the operands' signs (Inf and NaN as they are) instead
    auto walk = [&](auto plain) __attribute__((always_inline)) {
#pragma unroll
        for (int ob = 0; ob < CS_OB; ++ob)
#pragma unroll
            for (int t = 0; t < 9; ++t) acc[ob][t] = (v4f){0.f, 0.f, 0.f, 0.f};

        // the chunk being multiplied (c), the next (n): group of core channels and chunk of rows
        const int ig0 = ch_beg / pl.nyc;
        int c_i = ig0 * pl.ni, c_y = ch_beg - ig0 * pl.nyc;
        auto advance = [&](int& i, int& y) __attribute__((always_inline)) {
            if (++y == pl.nyc) { y = 0; i += pl.ni; }
        };
        int n_i = c_i, n_y = c_y;
        // the first loads of Z, then (the table is complete) of G1; the buffers are cleared while they are on their way
        if (ch_beg < ch_end) fetch_z(c_i, c_y);
        // entry of a position group: slab offset of its window origin, byte offset of its G1 values, (core channel, row), positions
        for (int e = tid; e < 4 * pl.nk; e += CS_NT) {
            const int per = pl.ry * pl.ow, ii = e / per, rem = e - ii * per, yl = rem / pl.ow, ox = rem - yl * pl.ow;
            const bool in = ii < pl.ni;
            const int left = g.Wo - 8 * ox;
            tab[e] = in ? make_int4(ii * pl.zi + yl * g.sh * pl.px + 8 * ox, 4 * (ii * g.cout * HoWo + yl * g.Wo + 8 * ox), (ii << 16) | yl, left < 8 ? left : 8)
                        : make_int4(0, 0, 0xffff, 0);
        }
        __syncthreads();
        if (ch_beg < ch_end && kgrp < pl.nk) fetch_a(c_i, c_y, kgrp);
        for (int e = tid; e < bufsz / 4; e += CS_NT) reinterpret_cast<uint4*>(buf)[e] = make_uint4(0u, 0u, 0u, 0u);   // both buffers
        __syncthreads();
        if (ch_beg < ch_end) {
            store_z(buf, plain);
            advance(n_i, n_y);
        }
        if (ch_beg + 1 < ch_end) fetch_z(n_i, n_y);
        __syncthreads();
        const int khs = g.dh * pl.px;
#pragma unroll 1
        for (int ch = ch_beg; ch < ch_end; ++ch) {
            const int cur = (ch - ch_beg) & 1;
            const bool more = ch + 1 < ch_end;
            int f_i = n_i, f_y = n_y;
            if (more) {
                store_z(buf + (cur ^ 1) * bufsz, plain);
                if (ch + 2 < ch_end) {
                    advance(f_i, f_y);
                    fetch_z(f_i, f_y);
                }
            }
#pragma unroll 1
            for (int kb = kgrp; kb < pl.nk; kb += CS_KG) {
                // this K block's G1 as bf16 terms; the next one's is requested
                v4u a[CS_OB][3];
#pragma unroll
                for (int ob = 0; ob < CS_OB; ++ob)
#pragma unroll
                    for (int d = 0; d < 4; ++d) {
                        float x = __uint_as_float(araw[ob][d >> 1][2 * (d & 1)]), y = __uint_as_float(araw[ob][d >> 1][2 * (d & 1) + 1]);
                        if (RAGGED) {
                            x = 2 * d < a_left ? x : 0.f;
                            y = 2 * d + 1 < a_left ? y : 0.f;
                        }
                        unsigned h, m = 0, l = 0;
                        if constexpr (plain()) h = class_pair(x, y, &huge);
                        else split_pair(x, y, h, m, l);
                        a[ob][0][d] = h; a[ob][1][d] = m; a[ob][2][d] = l;
                    }
                const unsigned short* zb = buf + cur * bufsz + a_org + ll * pl.zj;
                if (kb + CS_KG < pl.nk) fetch_a(c_i, c_y, kb + CS_KG);
                else if (more) fetch_a(n_i, n_y, kgrp);
                constexpr int WD = SW == 1 ? 5 : 9;          // dwords of a window; stride two: five even, four odd
                unsigned w[2][3][WD];
                auto window = [&](int kh, unsigned (&d)[3][WD]) __attribute__((always_inline)) {
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        const unsigned short* zr = zb + t * pl.zt + kh * khs;
                        const v4u q = *reinterpret_cast<const v4u*>(zr);
                        d[t][0] = q[0]; d[t][1] = q[1]; d[t][2] = q[2]; d[t][3] = q[3];
                        d[t][4] = *reinterpret_cast<const unsigned*>(zr + 8);
                        if constexpr (SW == 2) {
                            const v4u o = *reinterpret_cast<const v4u*>(zr + (pl.px >> 1));
                            d[t][5] = o[0]; d[t][6] = o[1]; d[t][7] = o[2]; d[t][8] = o[3];
                        }
                    }
                };
                window(0, w[0]);
#pragma unroll
                for (int kh = 0; kh < 3; ++kh) {
                    if (kh < 2) window(kh + 1, w[(kh + 1) & 1]);
                    __builtin_amdgcn_sched_barrier(0);
                    const unsigned (&d)[3][WD] = w[kh & 1];
                    v4u b[3][3];                             // [tap of the row][term]
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        b[0][t] = (v4u){d[t][0], d[t][1], d[t][2], d[t][3]};
                        v4u next;                            // the window one entry on
#pragma unroll
                        for (int q = 0; q < 4; ++q) next[q] = __builtin_amdgcn_alignbit(d[t][q + 1], d[t][q], 16);
                        if constexpr (SW == 1) {
                            b[1][t] = next;
#pragma unroll
                            for (int q = 0; q < 4; ++q) b[2][t][q] = copy(d[t][q + 1]);
                        } else {
                            b[1][t] = (v4u){d[t][WD - 4], d[t][WD - 3], d[t][WD - 2], d[t][WD - 1]};
                            b[2][t] = next;
                        }
                    }
                    // small terms first; six accumulators take turns
                    constexpr int TA[6] = {2, 0, 1, 1, 0, 0}, TB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                    for (int p = plain() ? 5 : 0; p < 6; ++p)
#pragma unroll
                        for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                            for (int ob = 0; ob < CS_OB; ++ob) acc[ob][3 * kh + dx] = mfma_bf16(a[ob][TA[p]], b[dx][TB[p]], acc[ob][3 * kh + dx]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            c_i = n_i; c_y = n_y;
            n_i = f_i; n_y = f_y;
            __syncthreads();
        }

        // lane holds o = o0 + 16 (2 wo + ob) + 4 lg + v, j = j0 + ll.  The K groups add their tiles in LDS in a fixed order (groups 2
        // and 3 write two tiles, 0 and 1 add to them, the store adds the two), and for one output channel the (j, tap) values of
        // this workgroup are then one contiguous run of T.
        if (tid < 2) met[tid] = 0;
#pragma unroll
        for (int round = 0; round < 2; ++round) {
            if (kgrp >> 1 == 1 - round) {
                float* Tg = Ts + (kgrp & 1) * TS_SZ;
#pragma unroll
                for (int ob = 0; ob < CS_OB; ++ob)
#pragma unroll
                    for (int t = 0; t < 9; ++t)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            float* p = &Tg[(16 * (CS_OB * wo + ob) + 4 * lg + v) * CS_TS_LD + ll * 9 + t];
                            *p = round == 0 ? acc[ob][t][v] : *p + acc[ob][t][v];
                        }
            }
            __syncthreads();
        }
    };
    const long long total = (long long)g.cout * g.r2 * 9;
    const int nj = (g.r2 - j0 < 16) ? g.r2 - j0 : 16;
    const int rowlen = nj * 9;
    const float inv_rowlen = 1.0f / (float)rowlen;
    float* __restrict__ out = jb.Tpart + (long long)bz * total;
    // f(where in T, output channel, (j, tap), value of the tiles) for the entries that this thread stores
    auto entries = [&](auto f) __attribute__((always_inline)) {
        for (int e = tid; e < CR_TO * rowlen; e += CS_NT) {              // e < 9216: the rounded float quotients are exact
            const int ol = (int)(((float)e + 0.5f) * inv_rowlen), c = e - ol * rowlen, o = o0 + ol;
            if (o < g.cout) f(out + ((long long)o * g.r2 + j0) * 9 + c, o, c, Ts[ol * CS_TS_LD + c] + Ts[TS_SZ + ol * CS_TS_LD + c]);
        }
    };
    walk(std::false_type());
    bool special = false;
    entries([&](float* t, int, int, float v) __attribute__((always_inline)) {
        *t = v;
        special = special || !(fabsf(v) < INFINITY);
    });
    if (special) met[0] = 1;
    wait_copies_and_sync<32>();                          // (for the flags, not for the stores)
    if (met[0] == 0) return;                             // (the same for all threads)
    __syncthreads();
    // Entries that are not finite: a term product of Inf and 0 is NaN, also where the product of the values is Inf, and an infinite value
    // has no further terms.  A second walk over signs tells what plain sums would be, NaN, Inf or finite, in the time of the first (a gradient
    // that is NaN throughout is what loss scaling makes now and then; the weight gradient of 256 x 48 x 9 over 8 x 64 x 64, finite 74 us, took
    // 4.8 ms entry by entry, 110 us so).
    walk(std::true_type());
    if (huge) met[0] = 1;
    if (z_special) met[1] = 1;
    __syncthreads();
    const bool any_huge = met[0] != 0, any_z = met[1] != 0;
    entries([&](float* t, int o, int c, float what) __attribute__((always_inline)) {
        if (fabsf(*t) < INFINITY) return;
        const bool finite = fabsf(what) < INFINITY;
        if (!finite) *t = what;
        // left: sums of finite values that overflow; a value that rounds to an infinite bf16 one; and zeros in the place of positions that
        // there are not, times an infinite entry of Z.  The latter two again as plain sums.
        if (finite ? !any_huge : !any_z) return;
        const int jl = (int)(((float)c + 0.5f) * (1.0f / 9.0f)), tap = c - 9 * jl, kh = tap / 3, kw = tap - 3 * kh;
        float v = 0.f;
        for (int ch = ch_beg; ch < ch_end; ++ch) {
            const int ig = ch / pl.nyc, y0 = (ch - ig * pl.nyc) * pl.ry, y1 = min(y0 + pl.ry, g.Ho);
            const int i1 = min((ig + 1) * pl.ni, g.r1);
            for (int i = ig * pl.ni; i < i1; ++i)
                for (int y = y0; y < y1; ++y) {
                    const int yy = y * g.sh - g.ph + kh * g.dh;
                    if (yy < 0 || yy >= g.H || isnan(v)) continue;
                    const float* gp = G1 + ((long long)i * g.cout + o) * HoWo + (long long)y * g.Wo;
                    const float* zp = Z + ((long long)i * g.r2 + j0 + jl) * HW + (long long)yy * g.W;
                    for (int x = 0; x < g.Wo; ++x) {
                        const int xx = x * SW - g.pw + kw;
                        if (xx >= 0 && xx < g.W) v = fmaf(gp[x], zp[xx], v);
                    }
                }
        }
        *t = v;
    });
}

template <bool RAGGED, int SW>
static hipError_t launch_split(const Batch<CorrJob>& b, dim3 grid, size_t lds, hipStream_t st) {
    static LdsAllowed allowed;
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_corr_mfma_split<9, RAGGED, SW>), CS_LDS_MAX, allowed);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_corr_mfma_split<9, RAGGED, SW>), grid, CS_NT, lds, st, b);
    return hipGetLastError();
}
// (the layers of a launch have one stride along W)
hipError_t launch_corr_split(const Batch<CorrJob>& b, dim3 grid, hipStream_t st) {
    size_t lds = 0;
    bool ragged = false;
    for (int j = 0; j < b.njobs; ++j) {
        lds = split_lds(b.job[j].pl) > lds ? split_lds(b.job[j].pl) : lds;
        ragged = ragged || b.job[j].g.Wo % 8 != 0;
    }
    if (b.job[0].g.sw == 2) return ragged ? launch_split<true, 2>(b, grid, lds, st) : launch_split<false, 2>(b, grid, lds, st);
    return ragged ? launch_split<true, 1>(b, grid, lds, st) : launch_split<false, 1>(b, grid, lds, st);
}

}  // namespace asi
