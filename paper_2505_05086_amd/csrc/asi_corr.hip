// Step 4 of Eq. 14 on fp32 MFMA (3 x 3 taps with a stride of one or two and unit dilation along W: asi_corr_split.hip):
//     T[o,j,kh,kw] = sum_{i,y,x} G1[i,o,y,x] * Zpad[i,j, y*s - p + kh*d, x*s - p + kw*d]
// an implicit GEMM with M = cout (o), N = (tap, j), K = (i, y, x).  A workgroup owns 64
// output channels x 16 core channels j x all taps and walks its share of K in chunks of one
// core channel i and up to 64 output positions (whole output rows).  Per chunk it stages
//   As[k][o]           the G1 tile, so that lane (o = l%16, k = l/16) reads its A operand
//   Zs[j][row][col]    the slab of Z rows the chunk touches, with a zero halo for the padding
// and for every tap the B operand of lane (k = l/16, j = l%16) is the slab entry of core channel j
// at the window origin of position k plus the tap's offset.
// Splits of K write partial T's that a reduction kernel sums in fixed order.
#include "asi_corr.h"
#include "asi_device.h"
#include "asi_lds.h"

#include <cstdio>
#include <cstring>
#include <type_traits>

namespace asi {

typedef float v4f __attribute__((ext_vector_type(4)));

// Output positions per chunk and the floats of LDS for the Z slab that goes with them, in one of two buffers: every wave stores
// the next chunk, issues the loads of the one after it and multiplies the current one, and a chunk costs one barrier.
// Slabs of up to CR_ZMAX_SHORT floats (7 x 7 with a halo: 16 x 81) have an instantiation of their own, whose loader takes half
// the loads.
constexpr int CR_KC = 64, CR_ZMAX_LONG = 4096, CR_ZMAX_SHORT = 2048;
// Waves per workgroup: 4 own 16 output channels each; with 8 the second four take every other
// K step of a chunk on accumulators of their own (summed through LDS at the end).  One wave per
// SIMD cannot overlap its operand reads and address arithmetic with its products (a step costs
// their sum, ~55-63 cycles per MFMA against 32); two waves per SIMD fill each other's gaps.
constexpr int CR_NW = 8;
constexpr int CR_NT = 64 * CR_NW;
constexpr int CR_KG = CR_NW / 4;     // K-step groups

// instantiation for a plan: low nibble 0 = <1,true,V>, 1 = <9,true,V>, 2 = <9,false,V>, 3 = <25,false,V>, V = the high nibble: 1 for
// short slabs; 0x100 the split-bf16 form, 0x101 with a stride of two along W
static unsigned corr_plan_key(const CorrGeom& g, const CorrPlan& p) {
    if (p.split) return g.sw == 2 ? 0x101u : 0x100u;
    const int taps = g.kh * g.kw;
    return (taps == 1 ? 0u : (taps == 9 ? 1u : (taps < 9 ? 2u : 3u))) | (p.zld * 16 <= CR_ZMAX_SHORT ? 0x10u : 0u);
}

// The plan of a layer that has the launch to itself.  cut: its chunks are dealt out by the rule for long walks.
static bool corr_plan(const CorrGeom& g, CorrPlan* p, bool* cut) {
    if (corr_split_plan(g, p, cut)) return true;
    std::memset(p, 0, sizeof(*p));
    const int taps = g.kh * g.kw;
    if (g.Wo > CR_KC || taps > 25) return false;
    // the kernel indexes G1 and Z with 32-bit offsets
    if ((long long)g.r1 * g.cout * g.Ho * g.Wo >= (1LL << 31) || (long long)g.r1 * g.r2 * g.H * g.W >= (1LL << 31)) return false;
    p->ry = CR_KC / g.Wo;
    if (p->ry > g.Ho) p->ry = g.Ho;
    p->wp = (g.Wo - 1) * g.sw + (g.kw - 1) * g.dw + 1;
    // fewer rows per chunk where a stride or a dilation makes the slab of Z that goes with them too large for LDS (a 45 x 37
    // map at stride 2, 101 channels, fell to the one-thread-per-output kernel: 117 us, 16 with chunks of two rows)
    while (p->ry > 1 && (long long)((p->ry - 1) * g.sh + (g.kh - 1) * g.dh + 1) * p->wp * 16 > CR_ZMAX_LONG) --p->ry;
    p->nyc = (g.Ho + p->ry - 1) / p->ry;
    p->rows_in = (p->ry - 1) * g.sh + (g.kh - 1) * g.dh + 1;
    p->slab = p->rows_in * p->wp;
    if ((long long)p->slab * 16 > CR_ZMAX_LONG) return false;
    // In the multiply loop lane (j = l%16, k = l/16) reads slab j at the window origin of position k,
    // and the positions of a lane group are sw floats apart.  With unit stride a slab pitch of
    // 2 mod 32 puts the 32 lanes of a half wave on 32 different banks (a pitch that is a multiple
    // of 32, e.g. 6 rows x 16 columns, puts the 16 slabs on one bank); otherwise an odd pitch.
    p->zld = p->slab;
    while (g.sw == 1 ? (p->zld % 32 != 2) : (p->zld % 2 == 0)) ++p->zld;
    if ((long long)p->zld * 16 > CR_ZMAX_LONG) p->zld = p->slab;
    p->nchunks = g.r1 * p->nyc;
    const long long base = corr_plan_tiles(g);
    long long target = 256;
    // Splits for one workgroup per CU, rounded down.  The 25-tap form fits a CU once (registers), so a workgroup beyond the
    // 256th waits for a whole round.  The others fit two or three times, but a workgroup's
    // first loads and its result, and the partial sums of the next launch, cost more than a second one per CU hides.  Splits
    // (the 3 x 3 ones measured before they had a form of their own) for 256 | 512 workgroups, correlation + expansion: 960 x 40 x 9 over 24 x 7 x 7 29 + 6 | 32 + 6 us, 256 x 32 x 9 over
    // 16 x 14 x 14 19 + 11 | 21 + 13, 320 x 40 x 1 over 24 x 7 x 7 8.7 + 9.3 | 8.7 + 10.6, 64 x 16 x 9 over 8 x 50 x 50
    // 19 + 17 | 21 + 26 (768: as 512 or slower).
    long long want = target / base;
    if (want > p->nchunks) want = p->nchunks;
    if (want < 1) want = 1;
    p->cps = (int)((p->nchunks + want - 1) / want);
    // A chunk is a dependent round of loads, a barrier and products: a workgroup that walks a thousand output positions or more
    // this way is cut in three, so that the workgroups of a CU (three with one tap, two with up to nine) hide each other's
    // rounds.  Correlation + expansion of the partial sums, cut | not cut: 1024 x 64 x 1 over 32 x 14 x 14 36 + 16 | 48 + 14 us;
    // 512 x 64 x 9 over 16 x 30 x 30 122 + 25 | 129 + 20, 768 over 32 x 13 x 13 86 + 33 | 94 + 27; with more channels still the
    // partial sums cost more than the overlap gains (1024 over 32 x 14 x 14 117 + 48 | 119 + 35).  The 25-tap form fits a CU
    // once (222 registers) and is cut for its sums: 512 x 64 x 25 over 16 x 28 x 28 would take 360 + 8 us instead of 413 + 16,
    // but three times as many of its additions would then be in fp32 (weight gradient off by 5.9e-7 instead of 3.9e-7).
    *cut = (long long)p->cps * p->ry * g.Wo >= 1024;
    if (*cut) {
        want = (3 * target + base - 1) / base;
        if (want > p->nchunks) want = p->nchunks;
        p->cps = (int)((p->nchunks + want - 1) / want);
    }
    p->nsplit = (p->nchunks + p->cps - 1) / p->cps;
    return true;
}

// The plan of layer `self` of a launch.  The layers share the CUs, and a workgroup costs about four chunks beside its own (first
// loads, result through LDS): every layer takes as many chunks per workgroup as give the fewest rounds x (chunks + 4) over
// the whole launch, never more splits than alone (three layers of 512 x 48 x 9 over 16 x 7 x 7 in the fp32 form, which they had then: 576
// workgroups of two chunks 46 us, 216 of six 32).  The split form's chunks hold up to 256 groups of positions and differ by layer, but a layer
// has few of them alone (eight of the 7 x 7 one) and the rule leaves little to choose: with one or twelve chunks in the place of the
// four, nine mixes of 7 x 7 to 64 x 64 layers took the same times (three 7 x 7 21.8 to 21.9 us, 7 x 7 beside 14 x 14 23.2 to 23.3, with
// 28 x 28 40.5 to 41.0, four 14 x 14 24.0 to 24.2).
static bool corr_plan_shared(const CorrGroup& grp, int self, CorrPlan* p) {
    bool cut;
    if (!corr_plan(*grp.g[self], p, &cut)) return false;
    if (grp.n <= 1 || cut) return true;
    CorrPlan pl[kMaxBatch];
    bool fixed[kMaxBatch];
    for (int k = 0; k < grp.n; ++k)
        if (!corr_plan(*grp.g[k], &pl[k], &fixed[k])) return false;
    long long best = -1;
    const int alone = p->nsplit;
    for (int ns = 1, last = 0; ns <= alone; ++ns) {
        const int cps = (p->nchunks + ns - 1) / ns;
        if (cps == last) continue;
        last = cps;
        long long wgs = 0;
        for (int k = 0; k < grp.n; ++k) {
            const int splits = (pl[k].nchunks + cps - 1) / cps;
            wgs += corr_plan_tiles(*grp.g[k]) * (fixed[k] || splits > pl[k].nsplit ? pl[k].nsplit : splits);
        }
        const long long cost = (wgs + 255) / 256 * (cps + 4);
        if (best < 0 || cost < best) { best = cost; p->cps = cps; }
    }
    p->nsplit = (p->nchunks + p->cps - 1) / p->cps;
    return true;
}


extern __shared__ float cr_dyn[];

template <int MAXT>
constexpr int corr_lds_floats(int kc, int zmax) {
    // two buffers of (G1 tile, Z slabs), then the table of window origins; afterwards the result tile
    return (CR_TO * (16 * (MAXT < 9 ? MAXT : 9) + 1) > 2 * (kc * (CR_TO + 1) + zmax) + kc)
               ? CR_TO * (16 * (MAXT < 9 ? MAXT : 9) + 1)
               : 2 * (kc * (CR_TO + 1) + zmax) + kc;
}
// SHORT: slabs of up to CR_ZMAX_SHORT floats
template <int MAXT, bool EXACT, bool SHORT>
__global__ __launch_bounds__(CR_NT) void k_corr_mfma(Batch<CorrJob> bt) {
    constexpr int CR_ZMAX = SHORT ? CR_ZMAX_SHORT : CR_ZMAX_LONG;
    constexpr int NWO = 4;                               // waves side by side along the output channels
    constexpr int KG = CR_KG;                            // K groups: waves that share channels and split the K steps
    // As | Zs | korg during the K loop; afterwards the 64 x (16 x up to 9 taps) result tile
    constexpr int CR_TG = MAXT < 9 ? MAXT : 9;           // taps per pass of the result through LDS
    constexpr int CR_TS_LD = 16 * CR_TG + 1;
    float* lds_raw = cr_dyn;                             // corr_lds_floats<MAXT>(CR_KC, CR_ZMAX) floats
    int lb;
    const CorrJob& jb = bt.job[locate_xcd(bt, &lb)];     // the tiles of one split share its G1 rows and Z slabs
    const float* __restrict__ G1 = jb.G1;
    const float* __restrict__ Z = jb.Z;
    float* __restrict__ Tpart = jb.Tpart;
    const CorrGeom g = jb.g;
    const CorrPlan pl = jb.pl;
    const int bz = lb / (jb.gx * jb.gy), brem = lb - bz * (jb.gx * jb.gy), by = brem / jb.gx, bx = brem - by * jb.gx;
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6, wo = wid % NWO, lg = lane >> 4, ll = lane & 15;
    const int kgrp_s = __builtin_amdgcn_readfirstlane(wid / NWO);      // the same for a whole wave: a scalar
    const int taps = g.kh * g.kw;
    const int o0 = bx * CR_TO, j0 = by * 16, z = bz;
    const int HoWo = g.Ho * g.Wo;

    int tapofs[MAXT];
#pragma unroll
    for (int t = 0; t < MAXT; ++t) {
        const int kh = t / g.kw, kw = t - kh * g.kw;
        tapofs[t] = (t < taps) ? kh * g.dh * pl.wp + kw * g.dw : 0;
    }
    v4f acc[MAXT];
#pragma unroll
    for (int t = 0; t < MAXT; ++t) acc[t] = (v4f){0.f, 0.f, 0.f, 0.f};

    const int ch_beg = z * pl.cps;
    const int ch_end = (ch_beg + pl.cps < pl.nchunks) ? ch_beg + pl.cps : pl.nchunks;
    const int ztotal = 16 * pl.slab;
    const float inv_slab = 1.0f / (float)pl.slab, inv_wp = 1.0f / (float)pl.wp, inv_wo = 1.0f / (float)g.Wo;
    const int row_step = g.sh * pl.wp;
    // loads per thread and chunk
    constexpr int NA = CR_KC * CR_TO / CR_NT, NZ = CR_ZMAX / CR_NT;
    static_assert(NA <= 32 && NZ <= 32, "one mask bit per load");
    float a_t[NA], z_t[NZ];
    unsigned amask = 0, zmask = 0;     // which of the loaded values belong to the chunk (set by fetch, used by the next store)
    // Loads of one chunk into registers: the G1 tile (64 channels x kcv positions, contiguous along k)
    // and the Z slab with its zero halo (rows ylo.., columns -pw..).  Every load goes to an address
    // that is valid whatever the lane (a lane outside the tile or in the halo reads a clamped position)
    // and its result is only masked when it is stored to LDS: a load guarded by a test of its own is
    // compiled into a conditional block that waits for it, and the loads of a chunk would then run one
    // after the other instead of together.
    constexpr int BUF = CR_KC * (CR_TO + 1) + CR_ZMAX;   // floats of one buffer
    // What a thread's Z loads depend on is fixed but for the core channel i and the chunk's first row: the slab row
    // (row_z), the offset of (core channel j, column) inside core channel i's planes, the LDS address.  Row, column and core
    // channel are clamped one by one (no select between two address expressions, no 64-bit multiply-add: both make the
    // compiler wait for earlier loads).
    const int nzu = (ztotal + CR_NT - 1) / CR_NT;                         // loads a thread needs (uniform)
    int off_z[NZ], row_z[NZ], dst_z[NZ];
    unsigned fix_z = 0;                // the loads that belong to the tile, whatever the chunk's rows
#pragma unroll
    for (int u = 0; u < NZ; ++u) {
        const int e = u * CR_NT + tid;
        // e < 4096, slab <= 256: the rounded float quotient is exact, no integer division needed
        const int jl = (int)(((float)e + 0.5f) * inv_slab), rem = e - __mul24(jl, pl.slab);
        const int rr = (int)(((float)rem + 0.5f) * inv_wp), col = rem - __mul24(rr, pl.wp) - g.pw, j = j0 + jl;
        fix_z |= ((e < ztotal) & (j < g.r2) & (col >= 0) & (col < g.W)) ? (1u << u) : 0u;
        off_z[u] = min(j, g.r2 - 1) * g.H * g.W + min(max(col, 0), g.W - 1);
        row_z[u] = rr;
        dst_z[u] = e < ztotal ? e + jl * (pl.zld - pl.slab) : -1;
    }
    const int k_a = tid & (CR_KC - 1);
    int off_a[NA];
#pragma unroll
    for (int u = 0; u < NA; ++u) {
        const int o = o0 + tid / CR_KC + (CR_NT / CR_KC) * u;
        off_a[u] = (o < g.cout ? o : o0) * HoWo;
    }
    auto fetch = [&](int ch) __attribute__((always_inline)) {
        const int i = ch / pl.nyc, yc = ch - i * pl.nyc;
        const int y0 = yc * pl.ry;
        const int rows = (g.Ho - y0 < pl.ry) ? g.Ho - y0 : pl.ry;
        const int kcv = rows * g.Wo;
        const int ylo = y0 * g.sh - g.ph;
        const float* __restrict__ Zi = Z + (unsigned)(i * g.r2) * (unsigned)(g.H * g.W);       // uniform
        zmask = 0;
#pragma unroll
        for (int u = 0; u < NZ; ++u) {
            if (u < nzu) {             // uniform
                const int row = ylo + row_z[u], rowc = min(max(row, 0), g.H - 1);
                z_t[u] = Zi[(unsigned)(off_z[u] + __mul24(rowc, g.W))];
                zmask |= row == rowc ? (1u << u) : 0u;
            }
        }
        zmask &= fix_z;
        // G1 tile: lane k of a wave walks the positions, the rows (channels) are CR_NT / CR_KC apart
        const bool kin = k_a < kcv;
        const float* __restrict__ Gi = G1 + ((unsigned)(i * g.cout) * (unsigned)HoWo + (unsigned)(y0 * g.Wo));     // uniform
        amask = 0;
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            a_t[u] = Gi[(unsigned)(off_a[u] + (kin ? k_a : 0))];
            amask |= (kin & (o0 + tid / CR_KC + (CR_NT / CR_KC) * u < g.cout)) ? (1u << u) : 0u;
        }
    };
    auto store = [&](float* buf) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NA; ++u)
            buf[k_a * (CR_TO + 1) + tid / CR_KC + (CR_NT / CR_KC) * u] = ((amask >> u) & 1u) ? a_t[u] : 0.f;
        float* zb = buf + CR_KC * (CR_TO + 1);
#pragma unroll
        for (int u = 0; u < NZ; ++u)
            if (u < nzu && dst_z[u] >= 0) zb[dst_z[u]] = ((zmask >> u) & 1u) ? z_t[u] : 0.f;
    };
    // korg[k]: offset of the window origin of output position k inside a slab, (k / Wo) * sh * wp + (k % Wo) * sw
    // (0 for positions beyond the rows of a chunk; their A values are zero).  The same for every chunk.
    int* korg = reinterpret_cast<int*>(lds_raw + 2 * BUF);
    for (int k = tid; k < CR_KC; k += CR_NT) {
        const int yl = (int)(((float)k + 0.5f) * inv_wo), x = k - yl * g.Wo;     // k < 2^14: exact
        korg[k] = (yl < pl.ry) ? yl * row_step + x * g.sw : 0;
    }
    // per-lane constants of the operand reads: As[4 ks + lg][16 wo + ll], slab ll of Zs
    const int a_lane = lg * (CR_TO + 1) + 16 * wo + ll, zlane = ll * pl.zld;
    auto chunk_positions = [&](int ch) __attribute__((always_inline)) {
        const int i = ch / pl.nyc, yc = ch - i * pl.nyc;
        const int y0 = yc * pl.ry;
        const int rows = (g.Ho - y0 < pl.ry) ? g.Ho - y0 : pl.ry;
        return rows * g.Wo;                                // valid positions in this chunk
    };
    // The products of one chunk held in LDS at (Ab, Zb).
    // Operands of step ks: one A value per channel block and one B value per tap.  The reads of step
    // ks + 1 are issued before the products of step ks, so that LDS latency is paid once per chunk
    // and not once per product.  Steps are taken in pairs; positions past the chunk's end have zero A
    // values (the loader's mask) and read the slab origin, so a step past the end adds nothing and the loop body stays free of
    // vector tests.
    // The step index is the same for a whole wave, so the A address is a per-lane constant plus a scalar,
    // and the window origin of a position comes from the table korg: no vector multiply is left in the
    // loop (besides their cost, the 64-bit multiply-add the compiler picks for some of them takes an
    // unrelated register - one of the next chunk's pending loads - as its unused upper addend and waits
    // for that load).
    auto multiply = [&](int kcv, const float* Ab, const float* Zb) __attribute__((always_inline)) {
        const int nsteps = (((kcv + 3) >> 2) + KG - 1) / KG;   // steps of this wave's K group: ks = kgrp, kgrp + KG, ...
        const int nst2 = (nsteps + 1) & ~1;
        int org = korg[4 * kgrp_s + lg];                   // origin of this lane's position in step 0
        auto operands = [&](int st, float& a, float (&bq)[MAXT]) __attribute__((always_inline)) {
            int ks = st * KG + kgrp_s;
            ks = ks < CR_KC / 4 ? ks : CR_KC / 4 - 1;          // only the read-ahead past the last step is clamped
            a = Ab[a_lane + ks * (4 * (CR_TO + 1))];           // positions past the chunk's end are zero
            const int zo = zlane + org;
#pragma unroll
            for (int t = 0; t < MAXT; ++t) bq[t] = (EXACT || t < taps) ? Zb[zo + tapofs[t]] : 0.f;
            int kn = ks + KG;
            kn = kn < CR_KC / 4 ? kn : CR_KC / 4 - 1;
            org = korg[4 * kn + lg];                           // for the next step of this wave
        };
        float a0, a1, b0[MAXT], b1[MAXT];
        operands(0, a0, b0);
        // (scheduling fences: left alone, the compiler moves each read down next to the product that uses
        // it, and the product then waits for the LDS round trip)
#pragma unroll 1
        for (int st = 0; st < nst2; st += 2) {
            operands(st + 1, a1, b1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < MAXT; ++t)
                if (EXACT || t < taps) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0, b0[t], acc[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            operands(st + 2, a0, b0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < MAXT; ++t)
                if (EXACT || t < taps) acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1, b1[t], acc[t], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    // two buffers: one barrier per chunk, and the loads of a chunk have the products of the one before to arrive
    // (one buffer, and the slab's index arithmetic done anew for every load and chunk: 30.0 us for 960 x 40 x 9 over
    // 24 x 7 x 7, 27.7 so)
    if (ch_beg < ch_end) {
        fetch(ch_beg);
        store(lds_raw);
    }
    if (ch_beg + 1 < ch_end) fetch(ch_beg + 1);
    __syncthreads();
#pragma unroll 1
    for (int ch = ch_beg; ch < ch_end; ++ch) {
        const int cur = (ch - ch_beg) & 1;
        const float* bcur = lds_raw + cur * BUF;
        if (ch + 1 < ch_end) store(lds_raw + (cur ^ 1) * BUF);
        if (ch + 2 < ch_end) fetch(ch + 2);
        multiply(chunk_positions(ch), bcur, bcur + CR_KC * (CR_TO + 1));
        __syncthreads();
    }
    // lane holds o = o0 + 16 wo + 4*lg + v, j = j0 + ll
    // The result goes through LDS, up to 9 taps at a time: the K groups add their tiles there, and
    // for one output channel the (j, tap) values of this workgroup are then one contiguous run of T
    // (stored straight from the accumulators every lane of a store would hit its own cache line:
    // the taps are innermost, lanes differ in j and o).
    const long long total = (long long)g.cout * g.r2 * taps;
    const int nj = (g.r2 - j0 < 16) ? g.r2 - j0 : 16;
    float* Ts = lds_raw;
#pragma unroll
    for (int t0 = 0; t0 < MAXT; t0 += CR_TG) {
        if (t0 < taps) {
            const int tg = (taps - t0 < CR_TG) ? taps - t0 : CR_TG;
            __syncthreads();                               // the tiles (or the previous pass) are no longer read
            // the K groups add their tiles in LDS in a fixed order
#pragma unroll
            for (int round = 0; round < KG; ++round) {
                if (kgrp_s == KG - 1 - round) {
#pragma unroll
                    for (int tt = 0; tt < CR_TG; ++tt)
                        if (t0 + tt < MAXT && tt < tg) {
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                float* p = &Ts[(16 * wo + 4 * lg + v) * CR_TS_LD + ll * tg + tt];
                                const float mine = acc[(t0 + tt < MAXT) ? t0 + tt : 0][v];
                                *p = (round == 0) ? mine : *p + mine;
                            }
                        }
                }
                __syncthreads();
            }
            const int rowlen = nj * tg;                    // <= 144
            const float inv_rowlen = 1.0f / (float)rowlen, inv_tg = 1.0f / (float)tg;
            for (int e = tid; e < CR_TO * rowlen; e += CR_NT) {   // e < 9216: the rounded float quotients are exact
                const int ol = (int)(((float)e + 0.5f) * inv_rowlen), c = e - ol * rowlen;
                const int jl = (int)(((float)c + 0.5f) * inv_tg), tt = c - jl * tg;
                const int o = o0 + ol;
                if (o < g.cout)
                    Tpart[(long long)z * total + ((long long)o * g.r2 + j0 + jl) * taps + t0 + tt] = Ts[ol * CR_TS_LD + c];
            }
        }
    }
}

// one thread per T[o,j,kh,kw] and split of the r1 axis: any geometry
__global__ __launch_bounds__(256) void k_corr(Batch<CorrJob> bt) {
    int lb;
    const CorrJob& jb = bt.job[locate(bt, &lb)];
    const float* __restrict__ G1 = jb.G1;
    const float* __restrict__ Z = jb.Z;
    float* __restrict__ Tpart = jb.Tpart;
    const CorrGeom g = jb.g;
    const int i_per_split = jb.ips;
    const int bsplit = lb / jb.gx, bx = lb - bsplit * jb.gx;
    const int taps = g.kh * g.kw;
    const long long total = (long long)g.cout * g.r2 * taps;
    const long long e = (long long)bx * 256 + threadIdx.x;
    if (e >= total) return;
    const int t = (int)(e % taps);
    const int j = (int)((e / taps) % g.r2);
    const int o = (int)(e / ((long long)taps * g.r2));
    const int kh = t / g.kw, kw = t - kh * g.kw;
    const int ibeg = bsplit * i_per_split;
    const int iend = (ibeg + i_per_split < g.r1) ? ibeg + i_per_split : g.r1;
    const int hoff = kh * g.dh - g.ph, woff = kw * g.dw - g.pw;
    float acc = 0.f;
    for (int i = ibeg; i < iend; ++i) {
        const float* g1p = G1 + ((long long)i * g.cout + o) * g.Ho * g.Wo;
        const float* zp = Z + ((long long)i * g.r2 + j) * g.H * g.W;
        for (int y = 0; y < g.Ho; ++y) {
            const int hh = y * g.sh + hoff;
            if (hh < 0 || hh >= g.H) continue;
            for (int x = 0; x < g.Wo; ++x) {
                const int ww = x * g.sw + woff;
                if (ww >= 0 && ww < g.W) acc = fmaf(g1p[y * g.Wo + x], zp[hh * g.W + ww], acc);
            }
        }
    }
    Tpart[(long long)bsplit * total + e] = acc;
}

bool corr_shares(const CorrGeom& a, const CorrGeom& b) {
    CorrPlan pa, pb;
    bool cut;
    return corr_plan(a, &pa, &cut) && corr_plan(b, &pb, &cut) && corr_plan_key(a, pa) == corr_plan_key(b, pb);
}

int corr_splits(const CorrGroup& grp, int self, CorrPlan* plan) {
    const CorrGeom& g = *grp.g[self];
    if (corr_plan_shared(grp, self, plan)) return plan->nsplit;
    plan->nsplit = 0;
    const long long total = (long long)g.cout * g.r2 * g.kh * g.kw;
    const long long blocks = (total + 255) / 256;
    long long want = (2048 + blocks - 1) / blocks;
    if (want > g.r1) want = g.r1;
    if (want < 1) want = 1;
    const int ips = (int)((g.r1 + want - 1) / want);
    return (g.r1 + ips - 1) / ips;
}

// key: see corr_plan_key; the fallback kernel has kind IT_CORR
bool make_corr(const float* G1, const float* Z, float* Tpart, const CorrGeom& g, const CorrPlan& plan, int nsplit, Item* out) {
    const long long total = (long long)g.cout * g.r2 * g.kh * g.kw;
    if (total <= 0 || nsplit <= 0 || !G1 || !Z || !Tpart) return false;
    CorrJob jb;
    std::memset(&jb, 0, sizeof(jb));
    jb.G1 = G1; jb.Z = Z; jb.Tpart = Tpart; jb.g = g;
    *out = Item();
    if (plan.nsplit > 0) {
        if (nsplit != plan.nsplit) return false;
        jb.pl = plan;
        jb.gx = (g.cout + CR_TO - 1) / CR_TO; jb.gy = (g.r2 + 15) / 16; jb.gz = jb.pl.nsplit;
        const int taps = g.kh * g.kw;
        out->kind = IT_CORR_MFMA;
        out->key = corr_plan_key(g, jb.pl);
        if (jb.pl.split) std::snprintf(out->label, sizeof(out->label), "k_corr_mfma_split<9, %s, %d>", g.Wo % 8 ? "true" : "false", g.sw);
        else std::snprintf(out->label, sizeof(out->label), "k_corr_mfma<%d, %s, %s>", taps == 1 ? 1 : (taps <= 9 ? 9 : 25),
                           (taps == 1 || taps == 9) ? "true" : "false", (out->key >> 4) ? "true" : "false");
    } else {
        jb.ips = (g.r1 + nsplit - 1) / nsplit;
        if ((total + 255) / 256 > 0x3fffffLL) return false;
        jb.gx = (int)((total + 255) / 256); jb.gy = nsplit; jb.gz = 1;
        out->kind = IT_CORR;
        std::snprintf(out->label, sizeof(out->label), "k_corr");
    }
    if ((long long)jb.gx * jb.gy * jb.gz > 0x3fffffffLL) return false;
    out->nblocks = jb.gx * jb.gy * jb.gz;
    static_assert(sizeof(CorrJob) <= kItemArgMax, "argument block");
    std::memcpy(out->arg, &jb, sizeof(jb));
    return true;
}

hipError_t launch_corr_items(const Item* const* items, int n, hipStream_t st) {
    Batch<CorrJob> b;
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    if (items[0]->kind == IT_CORR) {
        hipLaunchKernelGGL(k_corr, grid, 256, 0, st, b);
        return hipGetLastError();
    }
    if (items[0]->key >= 0x100u) return launch_corr_split(b, grid, st);
    // LDS is dynamic: most instantiations need more than the 64 KB a static array may take
#define ASI_CORR_LAUNCH(MAXT, EXACT, SHORT)                                                                        \
    do {                                                                                                           \
        constexpr size_t lds = sizeof(float) * corr_lds_floats<MAXT>(CR_KC, SHORT ? CR_ZMAX_SHORT : CR_ZMAX_LONG); \
        if (lds > 65536) {                                                                                         \
            static LdsAllowed allowed;                                                                             \
            const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_corr_mfma<MAXT, EXACT, SHORT>), lds, allowed); \
            if (e != hipSuccess) return e;                                                                         \
        }                                                                                                          \
        hipLaunchKernelGGL((k_corr_mfma<MAXT, EXACT, SHORT>), grid, CR_NT, lds, st, b);                            \
    } while (0)
    switch (items[0]->key) {
        case 0x0: ASI_CORR_LAUNCH(1, true, false); break;
        case 0x1: ASI_CORR_LAUNCH(9, true, false); break;
        case 0x2: ASI_CORR_LAUNCH(9, false, false); break;
        case 0x3: ASI_CORR_LAUNCH(25, false, false); break;
        case 0x10: ASI_CORR_LAUNCH(1, true, true); break;
        case 0x11: ASI_CORR_LAUNCH(9, true, true); break;
        case 0x12: ASI_CORR_LAUNCH(9, false, true); break;
        case 0x13: ASI_CORR_LAUNCH(25, false, true); break;
        default: return hipErrorInvalidValue;
    }
#undef ASI_CORR_LAUNCH
    return hipGetLastError();
}

}  // namespace asi
