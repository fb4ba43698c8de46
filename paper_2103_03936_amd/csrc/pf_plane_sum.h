// Sums over the planes of a channel (shift and bias gradients), shared by the kernels that form them.
#pragma once

#include "pf_common.h"

namespace pf {

__device__ __forceinline__ float plane_piece(const float *, const uint32_t (&w)[4])
{
    return (__uint_as_float(w[0]) + __uint_as_float(w[1])) + (__uint_as_float(w[2]) + __uint_as_float(w[3]));
}
__device__ __forceinline__ float plane_piece(const bf16_t *, const uint32_t (&w)[4])
{
    float e[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) e[k] = __uint_as_float(w[k] << 16) + __uint_as_float(w[k] & 0xffff0000u);
    return (e[0] + e[1]) + (e[2] + e[3]);
}

// The sum of channel c over N images [C][HW], 16-byte aligned, in all 256 threads, in a fixed order: planes of whole 16-byte pieces
// are read so, four in flight per thread.
template <typename T>
__device__ float plane_sum(const T *planes, int c, int N, int C, int HW)
{
    typedef unsigned int piece __attribute__((ext_vector_type(4), may_alias));
    constexpr int V = 16 / sizeof(T);
    const int tid = threadIdx.x;
    float acc = 0.f;
    if (HW % V == 0) {
        const int pv = HW / V;
        const i64 count = (i64)N * pv;
        for (i64 i0 = tid; i0 < count; i0 += 1024) {
            piece v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const i64 i = i0 + 256 * u < count ? i0 + 256 * u : count - 1;
                const int n = (int)(i / pv), q = (int)(i - (i64)n * pv);
                v[u] = *(const piece *)(planes + ((i64)n * C + c) * HW + (i64)q * V);
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
                const float s = plane_piece((const T *)nullptr, w);
                acc += i0 + 256 * u < count ? s : 0.f;
            }
        }
    } else {
        for (i64 i = tid; i < (i64)N * HW; i += 256) {
            const int n = (int)(i / HW), p = (int)(i - (i64)n * HW);
            acc += to_float(planes[((i64)n * C + c) * HW + p]);
        }
    }
    __shared__ float red[256];
    red[tid] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (tid < s) red[tid] += red[tid + s];
        __syncthreads();
    }
    return red[0];
}

} // namespace pf
