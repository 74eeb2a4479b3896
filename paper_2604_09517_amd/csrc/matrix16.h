// The 16 x 16 x 4 matrix instructions of the panel kernels, FP64 and FP32: lane
// (li, lq) = (lane % 16, lane / 16) supplies a = A[li][lq] and b = B[lq][li].
#pragma once

#include <hip/hip_runtime.h>

namespace {

template <typename T> struct Mat;
template <> struct Mat<double> {
    typedef double V4 __attribute__((ext_vector_type(4)));
    __device__ static V4 mul(double a, double b, V4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    __device__ static int row(int lq, int r) { return lq + 4 * r; }   // of accumulator r
};
template <> struct Mat<float> {
    typedef float V4 __attribute__((ext_vector_type(4)));
    __device__ static V4 mul(float a, float b, V4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    __device__ static int row(int lq, int r) { return 4 * lq + r; }
};

}  // namespace
