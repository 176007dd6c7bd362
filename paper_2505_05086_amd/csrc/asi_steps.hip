// Subspace steps of several modes of a layer in one launch: they all read the activation and nothing of each other, and each of
// them alone spends 5 to 7 us on its start, its first loads and the sums at its end.
//
// The bodies are those of the kernels that do one of them (asi_subspace_gram.h, asi_subspace_planes.h, asi_subspace_cols.h); a
// workgroup looks up whose it is.  8 x 32 x 16 x 16 (modes 8, 32 and 16 x 16 planes) 15.7 -> 6.6 us and two launches fewer, 64 x 256 x 14 x 14
// (64 and 14 x 14) 21.2 -> 18.4, three layers of 64 x 512 x 7 x 7 (64 and 7 x 7) 31.7 -> 29.2.
#include "asi_subspace_cols.h"
#include "asi_subspace_gram.h"
#include "asi_subspace_planes.h"

#include <cstdio>
#include <cstring>

namespace asi {

constexpr int ST_MAX = 3;
enum { ST_GRAM1, ST_GRAM2, ST_COLS, ST_PLANES1, ST_PLANES2, ST_TINY };
constexpr size_t st_arg_bytes() {
    size_t b = sizeof(GramJob);
    if (sizeof(ColsJob) > b) b = sizeof(ColsJob);
    if (sizeof(PlanesJob) > b) b = sizeof(PlanesJob);
    if (sizeof(TinyJob) > b) b = sizeof(TinyJob);
    return (b + 15) / 16 * 16;
}
struct StepsJob {
    int n, lds;                        // steps, bytes of LDS the largest needs
    int kind[ST_MAX], first[ST_MAX + 1];
    alignas(16) unsigned char arg[ST_MAX][st_arg_bytes()];
};

template <typename T>
__global__ __launch_bounds__(512, 4) void k_subspace_steps(Batch<StepsJob> bt) {
    int lb;
    const StepsJob& jb = bt.job[locate(bt, &lb)];
    int s = 0;
    while (s + 1 < jb.n && lb >= jb.first[s + 1]) ++s;
    lb -= jb.first[s];
    const unsigned char* arg = jb.arg[s];
    switch (jb.kind[s]) {
        case ST_GRAM1: subspace_gram<T, 1, true>(*reinterpret_cast<const GramJob*>(arg), lb); break;
        case ST_GRAM2: subspace_gram<T, 2, true>(*reinterpret_cast<const GramJob*>(arg), lb); break;
        case ST_COLS: {
            const ColsJob& cj = *reinterpret_cast<const ColsJob*>(arg);
            subspace_cols<T, true>(cj, xcd_order(lb, cj.nwg));
            break;
        }
        case ST_PLANES1: subspace_planes<T, 1, true>(*reinterpret_cast<const PlanesJob*>(arg), lb); break;
        case ST_PLANES2: subspace_planes<T, 2, true>(*reinterpret_cast<const PlanesJob*>(arg), lb); break;
        default: subspace_tiny<T, true>(*reinterpret_cast<const TinyJob*>(arg), lb); break;
    }
}

// kind, size of the argument block and LDS of a step that may share a launch; false for the others
static bool step_form(const Item& it, int* kind, size_t* bytes, int* lds) {
    const int nb = (int)((it.key >> 4) & 7u);
    if (!(it.key & 2u)) return false;                    // copied in single elements
    switch (it.kind) {
        case IT_GRAM_MODE:
            if (nb > 2) return false;
            *kind = nb == 1 ? ST_GRAM1 : ST_GRAM2; *bytes = sizeof(GramJob); *lds = nb == 1 ? sg_lds_bytes<1>() : sg_lds_bytes<2>();
            return true;
        case IT_SMALL:
            if (!(it.key & 4u)) return false;
            *kind = ST_COLS; *bytes = sizeof(ColsJob); *lds = SC_LDS;
            return true;
        case IT_PLANES: {
            if (nb > 2) return false;
            PlanesJob jb;
            std::memcpy(&jb, it.arg, sizeof(jb));
            *kind = nb == 1 ? ST_PLANES1 : ST_PLANES2; *bytes = sizeof(PlanesJob); *lds = jb.lds;
            return true;
        }
        case IT_TINY:
            *kind = ST_TINY; *bytes = sizeof(TinyJob); *lds = TY_RING * TY_BUF;
            return true;
    }
    return false;
}

// times that the chip is filled by this many workgroups
static long long fillings(long long blocks, int lds) {
    const long long resident = lds > 80 * 1024 ? 256 : 512;
    return (blocks + resident - 1) / resident;
}

// Appends `b` to the steps of `a`.  Where the Gram form of a mode is one of them its ring of buffers (96 KB) leaves room for one
// workgroup per CU, so it joins only where all workgroups of the layer are resident at once, and in a batch, whose layers' steps share the
// launch, where together they fill the chip no more often than apart (the columns and the planes fill it half as often there).
// Compress of 2 | 3 | 4 | 8 layers, apart -> all steps joined (fillings apart, joined): 16 x 32 x 20 x 20 (50 + 64 Gram, 128 planes) 31.7 -> 27.7 us (3, 2) |
// 35.5 -> 33.8 (3, 3) | 37.0 -> 39.5 (3, 4) | 56.8 -> 63.5 (6, 8); 8 x 32 x 32 x 32 (64 + 64, 64) 33.0 -> 27.6 | 34.5 -> 33.0 | 36.1 -> 36.3 (3, 3) |
// 55.5 -> 58.5 (5, 6); 32 x 64 x 14 x 14 (98 Gram, 52 columns) 34.6 -> 34.0 | 42.0 -> 37.6 | 46.0 -> 46.0 (3, 3) | 74.2 -> 72.2 (5, 5).  By the rule
// four and eight of the first take 37.0 and 57.7, eight of the second 57.6 (their Gram forms join).
bool join_steps(const Item& a, const Item& b, int layers, Item* out) {
    StepsJob jb;
    std::memset(&jb, 0, sizeof(jb));
    Item it = a;
    int kind, lds;
    size_t bytes;
    if (a.kind == IT_STEPS) {
        std::memcpy(&jb, a.arg, sizeof(jb));
    } else {
        if (!step_form(a, &kind, &bytes, &lds)) return false;
        jb.n = 1; jb.lds = lds; jb.kind[0] = kind; jb.first[1] = a.nblocks;
        std::memcpy(jb.arg[0], a.arg, bytes);
        it.kind = IT_STEPS; it.key = a.key & 1u;
        std::snprintf(it.label, sizeof(it.label), "k_subspace_steps<%s> = %s", (a.key & 1u) ? "asi::bf16_t" : "float", a.label);
    }
    if (jb.n >= ST_MAX || !step_form(b, &kind, &bytes, &lds) || (b.key & 1u) != (it.key & 1u)) return false;
    const int both = lds > jb.lds ? lds : jb.lds;
    const long long blocks = (long long)a.nblocks + b.nblocks, n = layers;
    if (blocks > 0x3fffffffLL || (both > 80 * 1024 && blocks > 256)) return false;
    if (fillings(n * blocks, both) > fillings(n * a.nblocks, jb.lds) + fillings(n * b.nblocks, lds)) return false;
    jb.lds = both;
    jb.kind[jb.n] = kind;
    std::memcpy(jb.arg[jb.n], b.arg, bytes);
    jb.first[++jb.n] = (int)blocks;
    it.nblocks = (int)blocks;
    const size_t len = std::strlen(it.label);
    std::snprintf(it.label + len, sizeof(it.label) - len, " + %s", b.label);
    it.bytes += b.bytes; it.flops += b.flops;
    static_assert(sizeof(StepsJob) <= kItemArgMax, "argument block");
    std::memcpy(it.arg, &jb, sizeof(jb));
    *out = it;
    return true;
}

template <typename T>
static hipError_t launch_steps_t(const Batch<StepsJob>& b, dim3 grid, int lds, hipStream_t st) {
    if (lds > 65536) {
        static LdsAllowed allowed;
        const hipError_t e = allow_lds(reinterpret_cast<const void*>(k_subspace_steps<T>), 160 * 1024, allowed);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((k_subspace_steps<T>), grid, 512, lds, st, b);
    return hipGetLastError();
}

hipError_t launch_steps_items(const Item* const* items, int n, hipStream_t st) {
    Batch<StepsJob> b;
    static_assert(sizeof(b) <= 4096, "kernel arguments");
    dim3 grid;
    if (!gather(items, n, &b, &grid)) return hipErrorInvalidValue;
    int lds = 0;
    for (int j = 0; j < n; ++j) lds = b.job[j].lds > lds ? b.job[j].lds : lds;
    return (items[0]->key & 1u) ? launch_steps_t<bf16_t>(b, grid, lds, st) : launch_steps_t<float>(b, grid, lds, st);
}

}  // namespace asi
