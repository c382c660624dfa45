// The 16 x 16 x 4 matrix-core products of the dense block kernels.  Operand lane
// layouts (checked on gfx950): lane l holds A[l % 16][l / 16] and
// B[l / 16][l % 16]; result value v of lane l is D[row(l, v)][l % 16].
#pragma once

#include <hip/hip_runtime.h>

namespace cast {

typedef double mf_v4d __attribute__((ext_vector_type(4)));
typedef float mf_v4f __attribute__((ext_vector_type(4)));

template <typename R> struct Mfma;
template <> struct Mfma<double> {
    using acc = mf_v4d;
    static __device__ __forceinline__ acc mma(double a, double b, acc c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return (lane >> 4) + 4 * v; }
};
template <> struct Mfma<float> {
    using acc = mf_v4f;
    static __device__ __forceinline__ acc mma(float a, float b, acc c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int v) { return 4 * (lane >> 4) + v; }
};

}  // namespace cast
