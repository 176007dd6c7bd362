// Plans and argument blocks that the correlation kernels share (asi_corr.hip, asi_corr_split.hip).
#pragma once
#include "asi_kernels.h"

namespace asi {

constexpr int CR_TO = 64;            // output channels per workgroup

struct CorrPlan {
    int split;       // 1: the split-bf16 form (asi_corr_split.hip), 0: the fp32 form
    int ry;          // output rows per chunk
    int nyc;         // chunks per core channel i (split form: per group of ni core channels)
    int rows_in;     // Z rows a chunk touches
    int wp;          // slab row length
    int nchunks;     // r1 * nyc (split form: ceil(r1 / ni) * nyc)
    int cps;         // chunks per split
    int nsplit;
    // fp32 form
    int slab;        // rows_in * wp
    int zld;         // floats between the slabs of consecutive core channels in LDS
    // split form, sizes in 16-bit elements
    int ni;          // core channels i per chunk
    int ow;          // groups of eight output positions per output row
    int nk;          // K blocks (four such groups) per chunk
    int px;          // slab row pitch (stride two: the even entries, then the odd ones)
    int zj, zi, zt;  // from one core channel j, core channel i, bf16 term to the next
};

struct CorrJob {
    const float* G1;
    const float* Z;
    float* Tpart;
    CorrGeom g;
    CorrPlan pl;
    int gx, gy, gz;      // channel tiles x core-channel tiles x splits (fallback kernel: blocks x splits x 1)
    int ips;             // fallback kernel: core channels i per split
};

inline long long corr_plan_tiles(const CorrGeom& g) { return (long long)((g.cout + CR_TO - 1) / CR_TO) * ((g.r2 + 15) / 16); }

// split form: chooses the chunk for a geometry that it takes (3 x 3 taps, a stride of one or two and unit dilation along W)
bool corr_split_plan(const CorrGeom& g, CorrPlan* p, bool* cut);
hipError_t launch_corr_split(const Batch<CorrJob>& b, dim3 grid, hipStream_t st);

}  // namespace asi
