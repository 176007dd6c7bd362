// Device code shared by the kernels that take a subspace step through a mode's Gram matrix (asi_gram.hip, asi_planes.hip).
//
// G (n x n, n <= 16 NB) is kept as its 16 x 16 blocks on and above the diagonal, block (mb, nb) at index
// mb NB - mb (mb - 1) / 2 + nb - mb, each in the order of the fp64 MFMA's result registers: element (i, j) of a block at
// (i / 4) 64 + (i % 4) 16 + j.
#pragma once
#include "asi_device.h"

namespace asi {

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

template <int NB>
constexpr int gram_blocks() { return NB * (NB + 1) / 2; }

// one K step (four indices) of G += X X^T: d[mb] holds element (row 16 mb + lane % 16, K slot lane / 16), for both sides
template <int NB>
__device__ __forceinline__ void gram_step(const double (&d)[NB][4], int s, v4d* acc) {
    int p = 0;
#pragma unroll
    for (int mb = 0; mb < NB; ++mb)
#pragma unroll
        for (int nb = mb; nb < NB; ++nb, ++p)
            acc[p] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[mb][s], d[nb][s], acc[p], 0, 0, 0);
}
template <int NB>
__device__ __forceinline__ void gram_put(const v4d* acc, double* dst, int lane) {
#pragma unroll
    for (int p = 0; p < gram_blocks<NB>(); ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v) dst[p * 256 + v * 64 + lane] = acc[p][v];
}
template <int NB>
__device__ __forceinline__ void gram_add(v4d* acc, const double* src, int lane) {
#pragma unroll
    for (int p = 0; p < gram_blocks<NB>(); ++p)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[p][v] += src[p * 256 + v * 64 + lane];
}

// P = G U (n x r) on the fp64 MFMA, a 16 x 16 block of P at a time; wave w of NW takes blocks w, w + NW, ..
// The first block's U may be requested early (gram_load_u) so that it arrives during the sums over the waves.
template <int NB>
__device__ __forceinline__ void gram_load_u(const float* __restrict__ U, int n, int r, int block, int lane, float (&u)[NB][4]) {
    const int lg = lane >> 4, q = 16 * (block / NB) + (lane & 15);
#pragma unroll
    for (int kb = 0; kb < NB; ++kb)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int k = 16 * kb + 4 * s + lg;
            u[kb][s] = U[(k < n && q < r) ? k * r + q : 0];
        }
}
template <int NB, int NW>
__device__ __forceinline__ void gram_times_u(const double* G, const float* __restrict__ U, int n, int r, double* __restrict__ out,
                                             int w, int lane, float (&u)[NB][4]) {
    const int lg = lane >> 4, ll = lane & 15, nblk = NB * ((r + 15) >> 4);
    for (int t = w; t < nblk; t += NW) {
        const int ib = t % NB, q = 16 * (t / NB) + ll;
        double ud[NB][4];
#pragma unroll
        for (int kb = 0; kb < NB; ++kb)
#pragma unroll
            for (int s = 0; s < 4; ++s) ud[kb][s] = (16 * kb + 4 * s + lg < n && q < r) ? (double)u[kb][s] : 0.0;
        if (t + NW < nblk) gram_load_u<NB>(U, n, r, t + NW, lane, u);
        if (16 * ib >= n) continue;
        v4d o = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kb = 0; kb < NB; ++kb) {
            if (16 * kb < n) {                         // uniform
                // block (ib, kb) of G: above the diagonal as stored, below it the transpose of (kb, ib)
                const int lo = ib < kb ? ib : kb, hi = ib < kb ? kb : ib;
                const double* g = G + (lo * NB - (lo * (lo - 1)) / 2 + hi - lo) * 256;
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const double x = ib < kb ? g[(ll >> 2) * 64 + (ll & 3) * 16 + 4 * s + lg] : g[s * 64 + lane];
                    o = __builtin_amdgcn_mfma_f64_16x16x4f64(16 * kb + 4 * s + lg < n ? x : 0.0, ud[kb][s], o, 0, 0, 0);
                }
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int i = 16 * ib + lg + 4 * v;
            if (i < n && q < r) out[i * r + q] = o[v];
        }
    }
}

// four consecutive elements from LDS, widened; vec: aligned for one read
__device__ __forceinline__ void read4(const float* p, bool vec, float (&x)[4]) {
    if (vec) {
        const v4f v = *reinterpret_cast<const v4f*>(p);
        x[0] = v[0]; x[1] = v[1]; x[2] = v[2]; x[3] = v[3];
    } else {
        x[0] = p[0]; x[1] = p[1]; x[2] = p[2]; x[3] = p[3];
    }
}
__device__ __forceinline__ void read4(const bf16_t* p, bool vec, float (&x)[4]) {
    if (vec) {
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        x[0] = __uint_as_float(v.x << 16); x[1] = __uint_as_float(v.x & 0xffff0000u);
        x[2] = __uint_as_float(v.y << 16); x[3] = __uint_as_float(v.y & 0xffff0000u);
    } else {
        x[0] = to_f32(p[0]); x[1] = to_f32(p[1]); x[2] = to_f32(p[2]); x[3] = to_f32(p[3]);
    }
}

}  // namespace asi
