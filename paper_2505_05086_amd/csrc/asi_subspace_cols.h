// Kernel body of the subspace step of modes of 49 to 64 entries (asi_subspace.hip), on its own so that a launch can do several modes' steps.
#pragma once
#include "asi_gram_device.h"
#include "asi_kernels.h"

namespace asi {

// ---- modes of 49 to 64 entries and up to 16 ranks over a long inner extent (asi_gram.hip takes the others) -----------------
// Nothing goes through LDS: a wave takes 16 consecutive columns and loads them twice, in the two layouts that its products want:
//   V (fp32 MFMA)  A operand (16 columns x 4 i):  row 4 s + lane / 16, column lane % 16           16 dwords
//   P (fp64 MFMA)  A operand (16 i x 4 columns):  row 16 mb + lane % 16, columns 4 (lane / 16) + v   4 pieces of four columns
// K slot (v, lane group) of the second product is column 4 lg + v, which is where the first product leaves V in register v.  The
// second set of loads meets the lines of the first in the L1.  U_prev is in registers, no wave waits for another before the
// sums at the end.  The form with a tile in LDS was bound by its loads, stores, reads and barriers (its products are 3 us):
// three 64 x 512 x 7 x 7 layers at rank 8 in one launch 23.0 -> 14.5 us, 64 x 256 x 14 x 14 at rank 16 14.6 -> 10.4
constexpr int SC_NT = 512, SC_NW = SC_NT / 64, SC_NB = 4, SC_LDS = SC_NW * SC_NB * 256 * 8;
extern __shared__ __align__(16) unsigned char sc_raw[];
struct ColsJob {
    const void* X;           // (outer, n, inner)
    const float* U;          // (n, r)
    double* part;            // (nwg, n, r)
    long long outer, inner, nblk;    // blocks of 16 columns
    int bpo;                 // blocks per outer slice
    int n, r, nwg;
    int32_t* zero;           // nullable: `nzero` int32 to clear
    int nzero;
};
template <typename T> struct ColsPiece { typedef v4f type; };
template <> struct ColsPiece<bf16_t> { typedef uint2 type; };
__device__ __forceinline__ v4f cols_widen(const v4f& p) { return p; }
__device__ __forceinline__ v4f cols_widen(const uint2& p) {
    return (v4f){__uint_as_float(p.x << 16), __uint_as_float(p.x & 0xffff0000u), __uint_as_float(p.y << 16), __uint_as_float(p.y & 0xffff0000u)};
}

// VEC: the inner extent is a multiple of four and X is aligned to four elements
template <typename T, bool VEC>
__device__ __forceinline__ void subspace_cols(const ColsJob& jb, int lb) {
    double (*red)[SC_NB * 256] = reinterpret_cast<double (*)[SC_NB * 256]>(sc_raw);
    const T* __restrict__ X = static_cast<const T*>(jb.X);
    const int n = jb.n, r = jb.r, tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, ll = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const long long inner = jb.inner, nblk = jb.nblk;
    if (jb.zero && lb == 0 && tid < jb.nzero) jb.zero[tid] = 0;
    const bool r_in = ll < r;
    // B operand of the first product: U[4 s + lg][ll]
    float u[4 * SC_NB];
#pragma unroll
    for (int s = 0; s < 4 * SC_NB; ++s) { const int i = 4 * s + lg; u[s] = jb.U[(i < n && r_in) ? i * r + ll : 0]; }
    v4d acc[SC_NB];
#pragma unroll
    for (int mb = 0; mb < SC_NB; ++mb) acc[mb] = (v4d){0.0, 0.0, 0.0, 0.0};
    // rows past the mode read the last one: masked in the first product, dropped in the second
    const long long lastrow = (long long)(n - 1) * inner;
    for (long long blk = (long long)lb * SC_NW + wave; blk < nblk; blk += (long long)jb.nwg * SC_NW) {
        const long long o = blk / jb.bpo, j0 = (blk - o * jb.bpo) * 16;
        const int left = (int)(inner - j0 < 16 ? inner - j0 : 16);           // columns of the block
        const T* __restrict__ xb = X + o * (long long)n * inner + j0;
        T xa[4 * SC_NB];
        typename ColsPiece<T>::type xv[SC_NB];
        T xs[VEC ? 1 : SC_NB][4];
        const long long ca = (long long)lg * inner + (ll < left ? ll : 0);
        const int c4 = 4 * lg < left ? 4 * lg : 0;
#pragma unroll
        for (int s = 0; s < 4 * SC_NB; ++s) xa[s] = 4 * s + 3 < 49 || 4 * s + lg < n ? xb[(long long)(4 * s) * inner + ca] : xb[lastrow + (ll < left ? ll : 0)];
#pragma unroll
        for (int mb = 0; mb < SC_NB; ++mb) {
            const long long row = 16 * mb + ll < n ? (long long)(16 * mb + ll) * inner : lastrow;
            if constexpr (VEC) xv[mb] = *reinterpret_cast<const typename ColsPiece<T>::type*>(xb + (row + c4));
            else
#pragma unroll
                for (int v = 0; v < 4; ++v) xs[mb][v] = xb[row + (4 * lg + v < left ? 4 * lg + v : 0)];
        }
        v4f vacc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < 4 * SC_NB; ++s) {
            const bool in = (4 * s + 3 < 49 || 4 * s + lg < n) && ll < left;
            const float a = in ? to_f32(xa[s]) : 0.f;
            const float b = (4 * s + 3 < 49 || 4 * s + lg < n) && r_in ? u[s] : 0.f;
            vacc = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, vacc, 0, 0, 0);
        }
        v4f x[SC_NB];
#pragma unroll
        for (int mb = 0; mb < SC_NB; ++mb) {
            if constexpr (VEC) {
                x[mb] = cols_widen(xv[mb]);
                if (4 * lg >= left) x[mb] = (v4f){0.f, 0.f, 0.f, 0.f};
            } else {
#pragma unroll
                for (int v = 0; v < 4; ++v) x[mb][v] = 4 * lg + v < left ? to_f32(xs[mb][v]) : 0.f;
            }
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const double b = (double)vacc[v];
#pragma unroll
            for (int mb = 0; mb < SC_NB; ++mb) acc[mb] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)x[mb][v], b, acc[mb], 0, 0, 0);
        }
    }
#pragma unroll
    for (int mb = 0; mb < SC_NB; ++mb)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][mb * 256 + 64 * v + lane] = acc[mb][v];
    __syncthreads();
    double* out = jb.part + (long long)lb * n * r;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int e = tid + SC_NT * h, i = 16 * (e >> 8) + ((e >> 4) & 3) + 4 * ((e >> 6) & 3), q = e & 15;      // fp64 MFMA result layout
        double s = red[0][e];
#pragma unroll
        for (int w = 1; w < SC_NW; ++w) s += red[w][e];
        if (i < n && q < r) out[i * r + q] = s;
    }
}

}  // namespace asi
