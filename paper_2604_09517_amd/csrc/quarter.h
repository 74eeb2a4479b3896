// Exchange between the four 16-lane quarters of a wave.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace {

// Value q of quarter wave b to quarter wave q, for each lane of the quarter.
template <int b>
__device__ __forceinline__ uint32_t spread32(uint32_t y0, uint32_t y1, uint32_t y2, uint32_t y3) {
    // rows (quarters) of p: y0's and y1's even ones, or odd ones
    const auto p = __builtin_amdgcn_permlane16_swap(y0, y1, false, false);
    const auto r = __builtin_amdgcn_permlane16_swap(y2, y3, false, false);
    return __builtin_amdgcn_permlane32_swap(p[b & 1], r[b & 1], false, false)[b >> 1];
}
template <int b>
__device__ __forceinline__ float spread(const float (&y)[4]) {
    return __uint_as_float(spread32<b>(__float_as_uint(y[0]), __float_as_uint(y[1]),
                                       __float_as_uint(y[2]), __float_as_uint(y[3])));
}
template <int b>
__device__ __forceinline__ double spread(const double (&y)[4]) {
    uint64_t u[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) u[i] = (uint64_t)__double_as_longlong(y[i]);
    const uint32_t lo = spread32<b>((uint32_t)u[0], (uint32_t)u[1], (uint32_t)u[2], (uint32_t)u[3]);
    const uint32_t hi = spread32<b>((uint32_t)(u[0] >> 32), (uint32_t)(u[1] >> 32),
                                    (uint32_t)(u[2] >> 32), (uint32_t)(u[3] >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

}  // namespace
