// Matrix-core types shared by the complex GEMM kernels (gfx950).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

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

// Map a linear workgroup id to (tile_m, tile_n).  Hardware dispatches
// consecutive ids round-robin over the 8 XCDs; regroup so that each XCD sees
// a contiguous run of ids (XCDs 0..r-1 take one tile more when the grid does
// not divide by 8).  Runs are then walked in groups of GM tile rows, M
// fastest: 32 consecutive tiles on one XCD cover 8 x 4 tiles, so A and B
// panels are both shared in that XCD's L2.
constexpr int64_t GM = 8;
__device__ inline void tile_of(int64_t bid, int64_t nbm, int64_t nbn, int64_t& tm, int64_t& tn) {
  const int64_t total = nbm * nbn;
  int64_t id = bid;
  if (total >= 64) {
    const int64_t q = total / 8, r = total % 8, x = bid % 8, j = bid / 8;
    id = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + j;
  }
  const int64_t width = GM * nbn;
  const int64_t first_m = (id / width) * GM;
  const int64_t gm = nbm - first_m < GM ? nbm - first_m : GM;
  const int64_t rem = id % width;
  tm = first_m + rem % gm;
  tn = rem / gm;
}

}  // namespace lrcc
