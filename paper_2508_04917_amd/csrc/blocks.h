// Device helpers of the setup kernels: workgroup scan, block arithmetic.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace ddilu {

__device__ __forceinline__ int wave_incl_scan(int v) {
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        int t = __shfl_up(v, d);
        if (lane >= d) v += t;
    }
    return v;
}

// Block-wide exclusive scan; sh must hold 65 ints; every thread must call.
__device__ __forceinline__ int block_excl_scan(int v, int *sh, int *total) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int inc = wave_incl_scan(v);
    if (lane == 63) sh[w] = inc;
    __syncthreads();
    int s = 0, si = 0;
    if (w == 0) {
        s = lane < nw ? sh[lane] : 0;
        si = wave_incl_scan(s);
    }
    __syncthreads();
    if (w == 0) {
        if (lane < nw) sh[lane] = si - s;
        if (lane == 63) sh[64] = si;
    }
    __syncthreads();
    *total = sh[64];
    int res = inc - v + sh[w];
    __syncthreads();
    return res;
}

// ------------------------------------------------------------ block math
template <int BS>
__device__ __forceinline__ void blk_mul(const double *A, const double *B, double *C) {
#pragma unroll
    for (int i = 0; i < BS; ++i)
#pragma unroll
        for (int j = 0; j < BS; ++j) {
            double s = 0.0;
#pragma unroll
            for (int k = 0; k < BS; ++k) s += A[i * BS + k] * B[k * BS + j];
            C[i * BS + j] = s;
        }
}

template <int BS>
__device__ __forceinline__ double blk_norm1(const double *A) {
    double m = 0.0;
#pragma unroll
    for (int j = 0; j < BS; ++j) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < BS; ++i) s += fabs(A[i * BS + j]);
        m = fmax(m, s);
    }
    return m;
}

// Inverse by the adjugate; false when the determinant vanishes, a value is
// not finite, or the 1-norm condition number exceeds 1e14.
template <int BS>
__device__ __forceinline__ bool blk_inverse(const double *a, double *inv) {
    if constexpr (BS == 1) {
        if (!(fabs(a[0]) > 0.0) || !isfinite(a[0])) return false;
        inv[0] = 1.0 / a[0];
        return true;
    } else {
        const double c00 = a[4] * a[8] - a[5] * a[7];
        const double c01 = a[5] * a[6] - a[3] * a[8];
        const double c02 = a[3] * a[7] - a[4] * a[6];
        const double det = a[0] * c00 + a[1] * c01 + a[2] * c02;
        if (!(fabs(det) > 0.0) || !isfinite(det)) return false;
        const double id = 1.0 / det;
        inv[0] = c00 * id;
        inv[1] = (a[2] * a[7] - a[1] * a[8]) * id;
        inv[2] = (a[1] * a[5] - a[2] * a[4]) * id;
        inv[3] = c01 * id;
        inv[4] = (a[0] * a[8] - a[2] * a[6]) * id;
        inv[5] = (a[2] * a[3] - a[0] * a[5]) * id;
        inv[6] = c02 * id;
        inv[7] = (a[1] * a[6] - a[0] * a[7]) * id;
        inv[8] = (a[0] * a[4] - a[1] * a[3]) * id;
        const double cond = blk_norm1<3>(a) * blk_norm1<3>(inv);
        return cond <= 1e14;
    }
}

}  // namespace ddilu
