// Wave-level pieces that several kernels share: the broadcast of a lane, and
// the 16x16x4 matrix-core product of a real type: operands A[lane % 16][lane /
// 16] and B[lane / 16][lane % 16], result element e of a lane at row
// row(lane, e), column lane % 16 (measured on gfx950).
#pragma once
#include <hip/hip_runtime.h>

namespace gwk {
namespace {

template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    typedef double v4 __attribute__((ext_vector_type(4)));
    static __device__ inline v4 op(double a, double b, v4 c) {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lane, int e) { return (lane >> 4) + 4 * e; }
};
template <>
struct Mfma<float> {
    typedef float v4 __attribute__((ext_vector_type(4)));
    static __device__ inline v4 op(float a, float b, v4 c) {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline int row(int lane, int e) { return 4 * (lane >> 4) + e; }
};

// v of lane k (uniform), in every lane.
__device__ inline double rlane(double v, int k) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, k), hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
__device__ inline float rlane(float v, int k) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), k)); }
__device__ inline int rlane(int v, int k) { return __builtin_amdgcn_readlane(v, k); }

}  // namespace
}  // namespace gwk
