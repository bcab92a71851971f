// Matrix-core types shared by the complex GEMM kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>

namespace lrcc {

typedef double d4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <typename T>
struct cpx;
// Output row of accumulator register r in lane group g = lane/16 (column
// lane%16): the FP64 instruction interleaves rows across lane groups, the
// FP32 one gives each lane group four consecutive rows.
template <>
struct cpx<double> {
  using type = double2;
  using acc = d4;
  static constexpr bool gauss = false;  // 4 real products
  static __device__ constexpr int row(int g, int r) { return g + 4 * r; }
};
template <>
struct cpx<float> {
  using type = float2;
  using acc = f4;
  static constexpr bool gauss = true;  // 3 real products
  static __device__ constexpr int row(int g, int r) { return 4 * g + r; }
};

__device__ inline d4 mfma(double a, double b, d4 c) { return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0); }
__device__ inline f4 mfma(float a, float b, f4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

}  // namespace lrcc
