// Output address map of the GEMM epilogue (device and host).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace lrcc {

// Output address map of a GEMM: element (m, n) of the product is stored at
// C + row(m) + col(n), with row(m) = sum_k digit_k(m) * mstr[k] over the
// mixed-radix digits of m (radices mdim[0..nm), the last varying fastest),
// and col(n) likewise.  This writes a product straight into a tensor whose
// index order interleaves the M and N indices (no permutation pass).
constexpr int kMapRank = 4;
struct OutMap {
  int nm = 1, nn = 1;
  int64_t mdim[kMapRank] = {1, 1, 1, 1}, mstr[kMapRank] = {0, 0, 0, 0};
  int64_t ndim[kMapRank] = {1, 1, 1, 1}, nstr[kMapRank] = {1, 0, 0, 0};
  static OutMap plain(int64_t ldc) {  // row-major with leading dimension ldc
    OutMap o;
    o.mstr[0] = ldc;
    o.mdim[0] = INT64_MAX;
    o.ndim[0] = INT64_MAX;
    return o;
  }
  __host__ __device__ static int64_t off(int64_t x, int nd, const int64_t* dim, const int64_t* str) {
    if (nd == 1) return x * str[0];
    int64_t o = 0;
    if (x < INT32_MAX) {  // 32-bit digit decode: far cheaper than 64-bit division on the GPU
      uint32_t y = (uint32_t)x;
      for (int k = nd - 1; k >= 0; --k) {
        const uint32_t dk = dim[k] > (int64_t)UINT32_MAX ? UINT32_MAX : (uint32_t)dim[k];
        const uint32_t q = y / dk;
        o += (int64_t)(y - q * dk) * str[k];
        y = q;
      }
      return o;
    }
    for (int k = nd - 1; k >= 0; --k) {
      const int64_t q = x / dim[k];
      o += (x - q * dim[k]) * str[k];
      x = q;
    }
    return o;
  }
  __host__ __device__ int64_t row(int64_t m) const { return off(m, nm, mdim, mstr); }
  __host__ __device__ int64_t col(int64_t n) const { return off(n, nn, ndim, nstr); }
  bool rows() const { return nm == 1 && nn == 1 && nstr[0] == 1; }  // a RowMap of mstr[0]
};

// Rows of ld elements, the layout of most products.  A kernel of its own type:
// with the digits of a DevMap in its arguments and epilogue the tiled kernel's
// main loop, compiled with fewer registers, ran up to 2 % longer (64 x 64 tile,
// mean of eight shapes: FP64 TN 1.9 %, 3000x3000x1500 1939 -> 1979 us; FP32 NT
// 1.7 %, the others 0.6 to 0.9 %).
struct RowMap {
  int64_t ld;
  __device__ int64_t row(int64_t x) const { return x * ld; }
  __device__ int64_t col(int64_t x) const { return x; }
};

// The map as the kernels take it.  An epilogue decodes some ten indices per
// lane; a 32-bit division by a run-time radix costs about 40 instructions, so
// each radix comes with its reciprocal (T. Granlund and P. L. Montgomery, PLDI
// 1994): q = (mulhi(y, mul) + y) >> sh for y < 2^31.  (FP32 into interleaved tensors, us with divisions -> so: 10800000 x
// 20 x 20 1380 -> 1212, 3600 x 60000 x 20 1283 -> 1107, 480 x 450000 x 20 1326
// -> 1152.)
struct DevMap {
  struct Side {
    int nd;
    uint32_t dim[kMapRank], mul[kMapRank], sh[kMapRank];
    int64_t str[kMapRank];
    __device__ int64_t off(int64_t x) const {
      if (nd == 1) return x * str[0];
      int64_t o = 0;
      uint32_t y = (uint32_t)x;
#pragma unroll
      for (int k = kMapRank - 1; k >= 0; --k) {
        if (k >= nd) continue;
        const uint32_t q = (__umulhi(y, mul[k]) + y) >> sh[k];
        o += (int64_t)(y - q * dim[k]) * str[k];
        y = q;
      }
      return o;
    }
  };
  Side m, n;
  __device__ int64_t row(int64_t x) const { return m.off(x); }
  __device__ int64_t col(int64_t x) const { return n.off(x); }

  static Side side(int nd, const int64_t* dim, const int64_t* str) {
    Side s{};
    s.nd = nd;
    for (int k = 0; k < nd; ++k) {
      s.str[k] = str[k];
      const uint64_t d = dim[k] < INT32_MAX ? (uint64_t)dim[k] : (uint64_t)INT32_MAX;
      uint32_t l = 0;
      while ((uint64_t(1) << l) < d) ++l;
      s.dim[k] = (uint32_t)d;
      s.mul[k] = (uint32_t)(((uint64_t(1) << 32) * ((uint64_t(1) << l) - d)) / d + 1);
      s.sh[k] = l;
    }
    return s;
  }
  // Indices stay below 2^31: the product of several radices is checked here
  // (a single radix is not decoded).
  static bool fits(const OutMap& o) {
    auto prod = [](int nd, const int64_t* dim) {
      double p = 1;
      for (int k = 0; k < nd; ++k) p *= (double)dim[k];
      return nd == 1 || p < 2147483648.0;
    };
    return prod(o.nm, o.mdim) && prod(o.nn, o.ndim);
  }
  explicit DevMap(const OutMap& o) : m(side(o.nm, o.mdim, o.mstr)), n(side(o.nn, o.ndim, o.nstr)) {}
};

}  // namespace lrcc
