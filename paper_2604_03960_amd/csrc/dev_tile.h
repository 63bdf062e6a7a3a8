// Device helpers of the kernels that keep tiles in registers: loops over compile-time indices and the
// 16 x 16 x 4 matrix instruction per operand type.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

namespace tna {

// f(integral_constant<int, B>) ... f(integral_constant<int, E - 1>): register arrays indexed by constants
template <int B, int E, class F>
__device__ __forceinline__ void static_for(F &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>{});
    static_for<B + 1, E>(f);
  }
}

// the same, ended by the first f that returns false: one jump past the rest of the code
template <int B, int E, class F>
__device__ __forceinline__ void static_while(F &&f) {
  if constexpr (B < E) {
    if (f(std::integral_constant<int, B>{})) static_while<B + 1, E>(f);
  }
}

typedef double v4d __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// 16 x 16 x 4 MFMA step and result layout per operand type.  Operands: A[i][k] in lane i + 16k,
// B[k][j] in lane j + 16k.  Result register r of lane group lk = lane / 16 holds row 4r + lk
// (f64) or 4lk + r (f32), column lane % 16.
template <class T> struct Mma;
template <> struct Mma<double> {
  typedef v4d acc;
  __device__ static acc step(double a, double b, acc c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
  __device__ static int row(int lk, int r) { return 4 * r + lk; }
};
template <> struct Mma<float> {
  typedef v4f acc;
  __device__ static acc step(float a, float b, acc c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
  __device__ static int row(int lk, int r) { return 4 * lk + r; }
};

}  // namespace tna
