// Steps 2 and 3 of Eq. 14, Z[p] = U3 S[p] U4^T for every plane p of the core, as device code: a wave takes 16 rows of a plane.
// Shared by k_z_planes and by the launches of G1, which carry it in extra workgroups (the two do not depend on each other).
#pragma once
#include "asi_device.h"

namespace asi {

struct ZPlanesJob {
    const float* S;      // (planes, r3, r4)
    const float* U3;     // (H, r3)
    const float* U4;     // (W, r4)
    float* Z;            // (planes, H, W)
    long long planes;
    int H, W, r3, r4;    // H, W <= 64, r3, r4 <= 32
    int hbs;             // waves of a plane: 1, 2 or 4
    int blocks;          // workgroups of four waves, 4 / hbs planes each
};

// Both products of a plane are a few thousand multiply-adds on operands that fit a wave's registers; as two mode
// products over the whole core they were two launches of 10 us each, bound by their round trips.  Here a wave takes rows
// h = 16 hb .. 16 hb + 15 of a plane: it loads the plane of S, its rows of U3 and the whole of U4 once
// and multiplies twice on the fp32 MFMA:
//   Z1^T[q, h] = sum_k S[k, q] U3[h, k]        A = S^T (row q = ll), B = U3^T (column h = ll)
//   Z^T[w, h]  = sum_q U4[w, q] Z1^T[q, h]     A = U4 (row w = ll),  B = Z1^T
// K slot lg of step s of a 16-block stands for index 16 block + 4 lg + s: a lane's B operand of the second product
// is then register s of the first product's result (row 4 lg + s of the block, column ll), so Z1 never leaves the
// registers, and the A operands are four consecutive indices.  The result registers hold four consecutive w of one row h.
// VEC: r3, r4 and W are multiples of four and all is aligned: 16-byte loads of the factors and stores.
// WB: blocks of 16 columns of the plane, all requested together; 0: any number, one after the other, for kernels that have no
// registers for more.
template <int WB, bool VEC>
__device__ __forceinline__ void z_plane_rows(const ZPlanesJob& jb, long long plane, int hb, int lane) {
    typedef float v4f __attribute__((ext_vector_type(4)));
    const int lg = lane >> 4, ll = lane & 15;
    const int H = jb.H, W = jb.W, r3 = jb.r3, r4 = jb.r4;
    const float* __restrict__ Sp = jb.S + plane * r3 * r4;

    // operands: all loads first, from addresses valid for every lane; masked afterwards
    constexpr int WN = WB ? WB : 1;
    v4f u3[2], u4[WN][2];
    float sa[2][2][4];
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
#pragma unroll
            for (int s_ = 0; s_ < 4; ++s_) {
                const int k = 16 * kb + 4 * lg + s_, q = 16 * qb + ll;
                sa[kb][qb][s_] = Sp[(k < r3 && q < r4) ? k * r4 + q : 0];
            }
    const int h = 16 * hb + ll;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
        const int k0 = 16 * kb + 4 * lg;
        if (VEC) u3[kb] = *reinterpret_cast<const v4f*>(jb.U3 + ((h < H && k0 < r3) ? h * r3 + k0 : 0));
        else
#pragma unroll
            for (int s_ = 0; s_ < 4; ++s_) u3[kb][s_] = jb.U3[(h < H && k0 + s_ < r3) ? h * r3 + k0 + s_ : 0];
    }
    auto load_u4 = [&](int w16) __attribute__((always_inline)) {
#pragma unroll
        for (int wb = 0; wb < WN; ++wb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                const int w = w16 + 16 * wb + ll, q0 = 16 * qb + 4 * lg;
                if (VEC) u4[wb][qb] = *reinterpret_cast<const v4f*>(jb.U4 + ((w < W && q0 < r4) ? w * r4 + q0 : 0));
                else
#pragma unroll
                    for (int s_ = 0; s_ < 4; ++s_) u4[wb][qb][s_] = jb.U4[(w < W && q0 + s_ < r4) ? w * r4 + q0 + s_ : 0];
            }
    };
    load_u4(0);
    const v4f zero4 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int s_ = 0; s_ < 4; ++s_) {
            const int k = 16 * kb + 4 * lg + s_;
            if (!VEC) u3[kb][s_] = (h < H && k < r3) ? u3[kb][s_] : 0.f;
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) sa[kb][qb][s_] = (k < r3 && 16 * qb + ll < r4) ? sa[kb][qb][s_] : 0.f;
        }
    if (VEC)
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) u3[kb] = (h < H && 16 * kb + 4 * lg < r3) ? u3[kb] : zero4;
    // Z1^T: z1[qb][e] = Z1^T[16 qb + 4 lg + e][16 hb + ll]
    v4f z1[2] = {zero4, zero4};
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
        if (16 * kb < r3)                                  // (uniform: a rank of at most 16 has one block)
#pragma unroll
            for (int s_ = 0; s_ < 4; ++s_)
#pragma unroll
                for (int qb = 0; qb < 2; ++qb)
                    z1[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(sa[kb][qb][s_], u3[kb][s_], z1[qb], 0, 0, 0);
    // Z^T: zt[wb][e] = Z[16 hb + ll][w16 + 16 wb + 4 lg + e]
    float* __restrict__ Zp = jb.Z + plane * H * W;
    auto columns = [&](int w16) __attribute__((always_inline)) {
        v4f zt[WN];
#pragma unroll
        for (int wb = 0; wb < WN; ++wb)
#pragma unroll
            for (int qb = 0; qb < 2; ++qb) {
                if (VEC) u4[wb][qb] = (w16 + 16 * wb + ll < W && 16 * qb + 4 * lg < r4) ? u4[wb][qb] : zero4;
                else
#pragma unroll
                    for (int s_ = 0; s_ < 4; ++s_) u4[wb][qb][s_] = (w16 + 16 * wb + ll < W && 16 * qb + 4 * lg + s_ < r4) ? u4[wb][qb][s_] : 0.f;
            }
#pragma unroll
        for (int wb = 0; wb < WN; ++wb) zt[wb] = zero4;
#pragma unroll
        for (int qb = 0; qb < 2; ++qb)
            if (16 * qb < r4)
#pragma unroll
                for (int s_ = 0; s_ < 4; ++s_)
#pragma unroll
                    for (int wb = 0; wb < WN; ++wb) zt[wb] = __builtin_amdgcn_mfma_f32_16x16x4f32(u4[wb][qb][s_], z1[qb][s_], zt[wb], 0, 0, 0);
#pragma unroll
        for (int wb = 0; wb < WN; ++wb) {
            const int w0 = w16 + 16 * wb + 4 * lg;
            if (VEC) {
                if (h < H && w0 < W) *reinterpret_cast<v4f*>(Zp + h * W + w0) = zt[wb];
            } else if (h < H) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (w0 + e < W) Zp[h * W + w0 + e] = zt[wb][e];
            }
        }
    };
    columns(0);
    if (WB == 0)
#pragma unroll 1
        for (int w16 = 16; w16 < W; w16 += 16) {
            load_u4(w16);
            columns(w16);
        }
}

// workgroup zb (four waves) of a job; no barrier
template <int WB, bool VEC>
__device__ __forceinline__ void z_planes_block(const ZPlanesJob& jb, int zb) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), hb = wave & (jb.hbs - 1);
    const long long plane = (long long)zb * (4 / jb.hbs) + wave / jb.hbs;
    if (plane < jb.planes && 16 * hb < jb.H) z_plane_rows<WB, VEC>(jb, plane, hb, threadIdx.x & 63);
}

}  // namespace asi
