// Matrix instructions by scalar type: v_mfma_f32_16x16x4_f32 and v_mfma_f64_16x16x4_f64.
// Both take A[i][k] from lane i + 16 k and B[k][j] from lane j + 16 k.
#pragma once

#include <hip/hip_runtime.h>

namespace mbd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename R> struct Mma;
template <> struct Mma<float> {
  typedef f32x4 acc;
  static __device__ __forceinline__ acc fma(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // matrix row of register r in a lane of row group g = lane / 16
  static __device__ __forceinline__ int row(int g, int r) { return 4 * g + r; }
};
template <> struct Mma<double> {
  typedef f64x4 acc;
  static __device__ __forceinline__ acc fma(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int g, int r) { return g + 4 * r; }
};

// N consecutive reals moved as one vector (at most 16 bytes).
template <typename R, int N>
struct alignas(sizeof(R) * N) Pack {
  R v[N];
};

}  // namespace mbd
