// Complex GEMM without LDS staging, for products with few or narrow tiles.
//
// The tiled kernel (gemm.hip) walks K one barrier-separated slab at a time; a
// slab takes 2.6 us when its workgroup has the CU to itself, so a product
// with a handful of tiles is bound by that chain and not by any rate of the
// chip (FP64 30 x 60 x 36000, split 34 ways: 190 us for 3 us of MFMA work
// and 11 us of memory traffic).  Here a wavefront loads the MFMA fragments
// of its 16 TI x 16 TJ tile straight from global memory, one step of 4 U
// depths ahead of the products, with no barrier in the loop:
//   KSPLIT   the NW wavefronts of a workgroup share one tile and take every
//            NW-th step each; their sums meet in LDS at the end.  Further
//            splits over blockIdx.y leave partials for splitk_reduce_kernel.
//   !KSPLIT  every wavefront owns a tile of its own (shallow products).
// Measured (us, tiled kernel -> this one): FP64 4x4x1024 170 -> 7, 3x600x600
// 102 -> 8, 180x10x6000 205 -> 15, 30x60x36000 190 -> 37, 135x1770x1770
// 295 -> 82, 1200^3 347 -> 257, 3000^3 3820 -> 3585, 20x450000x150 1141 ->
// 378, 1x22500x3000 859 -> 196 (5.5 TB/s); FP32 12x671x671 53 -> 7,
// 660x1830x1830 219 -> 150, 24x3000x3000 121 -> 34, 36000x1x3000 289 -> 155.
// Without LDS every operand element is read from L2 once per 32 rows or
// columns, which the FP32 3M products outrun when they are large and wide;
// those stay on the tiled kernel (wave_plan).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma.h"

namespace lrcc {

template <typename T, bool TA, bool TB, int TI, int TJ, int NW, bool KSPLIT, int U>
__global__ void __launch_bounds__(64 * NW)
    wgemm_kernel(int64_t M, int64_t N, int64_t K, T are, T aim, const typename cpx<T>::type* __restrict__ A,
                 int64_t lda, const typename cpx<T>::type* __restrict__ B, int64_t ldb, T bre, T bim,
                 typename cpx<T>::type* __restrict__ C, DevMap om, int64_t kchunk, int64_t cstride, T bsgn,
                 int64_t nbm) {
  using V2 = typename cpx<T>::type;
  using ACC = typename cpx<T>::acc;
  constexpr bool G3 = cpx<T>::gauss;
  constexpr int NA = G3 ? 3 : 2;
  constexpr int KS = 4 * U;  // depth of one step
  constexpr uint32_t ES = sizeof(V2);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  {
    const int64_t kbeg = (int64_t)blockIdx.y * kchunk;
    K = (K < kbeg + kchunk ? K : kbeg + kchunk) - kbeg;
    A += TA ? kbeg * lda : kbeg;
    B += TB ? kbeg : kbeg * ldb;
    C += (int64_t)blockIdx.y * cstride;
  }
  int64_t tile = blockIdx.x;
  if (!KSPLIT) {
    tile = tile * NW + wave;
    if (tile >= nbm * ((N + 16 * TJ - 1) / (16 * TJ))) return;
  }
  // Below 8192 tiles each XCD takes a run of neighbouring ones (FP64
  // 135x1770x1770 94 -> 88 us, 190x11175x11175 3590 -> 3480); longer grids
  // walk all rows of one column block together, so that the wide operand is
  // read once (1140x11175x11175 19400 us in runs, 18900 so).
  int64_t tm = tile % nbm, tn = tile / nbm;
  if (KSPLIT) {
    const int64_t nbn = (N + 16 * TJ - 1) / (16 * TJ);
    if (nbm * nbn < 8192) tile_of(tile, nbm, nbn, tm, tn);
  }
  const int64_t m0 = tm * (16 * TI), n0 = tn * (16 * TJ);

  // An operand address is a base common to the wavefront (advanced along k)
  // plus a 32-bit byte offset per lane.  Rows beyond M and columns beyond N
  // are clamped to the last one; they only feed outputs that are never stored.
  const char* ab = (const char*)(A + (TA ? m0 : m0 * lda));
  const char* bb = (const char*)(B + (TB ? n0 * ldb : n0));
  uint32_t oa[TI], ob[TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    const uint32_t r = i * 16 + r16, cr = m0 + r < M ? r : (uint32_t)(M - 1 - m0);
    oa[i] = (TA ? cr + kq * U * (uint32_t)lda : cr * (uint32_t)lda + kq * U) * ES;
  }
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const uint32_t r = j * 16 + r16, cr = n0 + r < N ? r : (uint32_t)(N - 1 - n0);
    ob[j] = (TB ? cr * (uint32_t)ldb + kq * U : cr + kq * U * (uint32_t)ldb) * ES;
  }
  const int64_t sa = (TA ? lda : 1) * ES, sb = (TB ? 1 : ldb) * ES;  // one depth, in bytes
  struct Frag {
    V2 a[U][TI], b[U][TJ];
  };
  // lane group kq holds the depths k0 + kq U + u of a step
  auto load = [&](Frag& f, int64_t k0) {
    const char* pa = ab + k0 * sa;
    const char* pb = bb + k0 * sb;
    if (k0 + KS <= K) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int i = 0; i < TI; ++i) f.a[u][i] = *(const V2*)(pa + u * sa + oa[i]);
#pragma unroll
        for (int j = 0; j < TJ; ++j) f.b[u][j] = *(const V2*)(pb + u * sb + ob[j]);
      }
    } else {  // depths beyond K are read at the last one and count as zero
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t kl = k0 + kq * U + u, back = kl < K ? 0 : kl - (K - 1);
#pragma unroll
        for (int i = 0; i < TI; ++i) {
          const V2 x = *(const V2*)(pa + u * sa + oa[i] - back * sa);
          f.a[u][i] = back ? V2{0, 0} : x;
        }
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          const V2 x = *(const V2*)(pb + u * sb + ob[j] - back * sb);
          f.b[u][j] = back ? V2{0, 0} : x;
        }
      }
    }
  };
  ACC acc[NA][TI][TJ];
#pragma unroll
  for (int p = 0; p < NA; ++p)
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j) acc[p][i][j] = ACC{0, 0, 0, 0};
  auto products = [&](const Frag& f) {
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j) {
          const V2 a = f.a[u][i], b = V2{f.b[u][j].x, f.b[u][j].y * bsgn};
          if constexpr (!G3) {
            acc[0][i][j] = mfma(a.x, b.x, acc[0][i][j]);
            acc[1][i][j] = mfma(a.x, b.y, acc[1][i][j]);
            acc[0][i][j] = mfma(-a.y, b.y, acc[0][i][j]);
            acc[1][i][j] = mfma(a.y, b.x, acc[1][i][j]);
          } else {
            acc[0][i][j] = mfma(a.x, b.x, acc[0][i][j]);
            acc[1][i][j] = mfma(a.y, b.y, acc[1][i][j]);
            acc[2][i][j] = mfma(a.x + a.y, b.x + b.y, acc[2][i][j]);
          }
        }
  };
  constexpr int64_t STEP = KSPLIT ? (int64_t)KS * NW : KS;
  int64_t k = KSPLIT ? (int64_t)wave * KS : 0;
  Frag f0, f1;
  if (k < K) load(f0, k);
  while (k < K) {
    if (k + STEP < K) load(f1, k + STEP);
    products(f0);
    k += STEP;
    if (k >= K) break;
    if (k + STEP < K) load(f0, k + STEP);
    products(f1);
    k += STEP;
  }
  auto value = [&](int i, int j, int r) {
    if constexpr (!G3) {
      return V2{acc[0][i][j][r], acc[1][i][j][r]};
    } else {
      const T p1 = acc[0][i][j][r], p2 = acc[1][i][j][r], p3 = acc[2][i][j][r];
      return V2{p1 - p2, p3 - p1 - p2};
    }
  };
  const bool use_beta = (bre != T(0) || bim != T(0));
  auto put = [&](int64_t off, V2 v) {
    T cr = are * v.x - aim * v.y, ci = are * v.y + aim * v.x;
    V2* c = C + off;
    if (use_beta) {
      const V2 y = *c;
      cr += bre * y.x - bim * y.y;
      ci += bre * y.y + bim * y.x;
    }
    *c = V2{cr, ci};
  };
  if constexpr (KSPLIT) {
    __shared__ V2 red[NW][TI * TJ * 256];
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          red[wave][(i * 16 + cpx<T>::row(kq, r)) * (16 * TJ) + j * 16 + r16] = value(i, j, r);
    __syncthreads();
    for (int e = tid; e < TI * TJ * 256; e += 64 * NW) {
      V2 s = red[0][e];
#pragma unroll
      for (int w = 1; w < NW; ++w) {
        s.x += red[w][e].x;
        s.y += red[w][e].y;
      }
      const int64_t m = m0 + e / (16 * TJ), n = n0 + e % (16 * TJ);
      if (m < M && n < N) put(om.row(m) + om.col(n), s);
    }
  } else {
    int64_t coff[TJ];
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      const int64_t n = n0 + j * 16 + r16;
      coff[j] = n < N ? om.col(n) : -1;
    }
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t m = m0 + i * 16 + cpx<T>::row(kq, r);
        if (m >= M) continue;
        const int64_t roff = om.row(m);
#pragma unroll
        for (int j = 0; j < TJ; ++j)
          if (coff[j] >= 0) put(roff + coff[j], value(i, j, r));
      }
  }
}

template <typename T, int TI, int TJ, int NW, bool KSPLIT, int U>
static void wgo(bool ta, bool tb, int64_t m, int64_t n, int64_t k, double are, double aim, const void* A, int64_t lda,
                const void* B, int64_t ldb, double bre, double bim, void* C, const OutMap& om, hipStream_t st,
                int splits, int64_t kchunk, int64_t cstride, bool conjb) {
  using V2 = typename cpx<T>::type;
  const int64_t nbm = (m + 16 * TI - 1) / (16 * TI), nt = nbm * ((n + 16 * TJ - 1) / (16 * TJ));
  const int64_t nb = KSPLIT ? nt : (nt + NW - 1) / NW;
  LRCC_REQUIRE(nb < (int64_t(1) << 31), LRCC_E_INVALID, "gemm grid too large");
#define WGO_(TA_, TB_)                                                                                           \
  hipLaunchKernelGGL((wgemm_kernel<T, TA_, TB_, TI, TJ, NW, KSPLIT, U>), dim3((unsigned)nb, (unsigned)splits),   \
                     dim3(64 * NW), 0, st, m, n, k, (T)are, (T)aim, (const V2*)A, lda, (const V2*)B, ldb, (T)bre, \
                     (T)bim, (V2*)C, DevMap(om), kchunk, cstride, (T)(conjb ? -1.0 : 1.0), nbm)
  if (!ta && !tb)
    WGO_(false, false);
  else if (!ta && tb)
    WGO_(false, true);
  else if (ta && !tb)
    WGO_(true, false);
  else
    WGO_(true, true);
#undef WGO_
  HIP_CHECK(hipGetLastError());
}

// Small products whose operands lie in any index order: element (m, k) of A
// lies at A + am(m) + ak(k), (n, k) of B at B + bn(n) + bk(k), so a small operand
// needs no permuted copy before its product.  One 16 x 16 tile per workgroup,
// K shared by its NW wavefronts as above; the offsets along K are decoded
// once per workgroup into LDS.  What bounds such a product is the latency of
// one pass (3-10 us by its depth, one or a few workgroups of 256 CUs busy), so
// up to kMapTerms products independent of each other share a launch.  Right
// product at o = 4, v = 16, FP64: 57 launches in 218 us alone, 33 in 161 in
// groups.
template <typename T>
struct MapTerm {
  using V2 = typename cpx<T>::type;
  struct Side {  // DevMap::Side with 32-bit strides: kernel arguments are limited to 4 KB
    uint32_t dim[kMapRank], mul[kMapRank];
    int32_t str[kMapRank];
    uint8_t sh[kMapRank];
    int nd;
    __device__ int off(int x) const {
      if (nd == 1) return x * str[0];
      int o = 0;
      uint32_t y = (uint32_t)x;
#pragma unroll
      for (int k = kMapRank - 1; k >= 0; --k) {
        if (k >= nd) continue;
        const uint32_t q = (__umulhi(y, mul[k]) + y) >> sh[k];
        o += (int)(y - q * dim[k]) * str[k];
        y = q;
      }
      return o;
    }
  };
  const V2 *A, *B;
  V2* C;
  T are, aim, beta;
  int M, N, K, nbm, k0;  // K depths from k0 on
  Side am, ak, bn, bk, cm, cn;
};
constexpr int kMapTerms = 8;
template <typename T>
struct MapGroup {
  int n, first[kMapTerms];  // first workgroup of each term
  MapTerm<T> t[kMapTerms];
};
static_assert(sizeof(MapGroup<double>) <= 3584, "kernel arguments: 4 KB with the implicit ones");

template <typename T, int NW>
__global__ void __launch_bounds__(64 * NW) mgemm_kernel(MapGroup<T> g) {
  using V2 = typename cpx<T>::type;
  using ACC = typename cpx<T>::acc;
  constexpr bool G3 = cpx<T>::gauss;
  constexpr int U = 4, KS = 4 * U, STEP = KS * NW;
  __shared__ uint32_t ka[kMapDepth], kb[kMapDepth];
  __shared__ V2 red[NW][256];
  int ti = 0;
#pragma unroll
  for (int i = 1; i < kMapTerms; ++i)
    if (i < g.n && (int)blockIdx.x >= g.first[i]) ti = i;
  const MapTerm<T>& p = g.t[ti];
  const int M = p.M, N = p.N, K = p.K, bid = (int)blockIdx.x - g.first[ti];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, kq = lane >> 4;
  const int m0 = (bid % p.nbm) * 16, n0 = (bid / p.nbm) * 16;
  for (int k = tid; k < K; k += 64 * NW) {
    ka[k] = (uint32_t)p.ak.off(p.k0 + k);
    kb[k] = (uint32_t)p.bk.off(p.k0 + k);
  }
  // rows beyond M and columns beyond N feed outputs that are never stored
  const V2* pa = p.A + p.am.off(m0 + r16 < M ? m0 + r16 : M - 1);
  const V2* pb = p.B + p.bn.off(n0 + r16 < N ? n0 + r16 : N - 1);
  __syncthreads();
  struct Frag {
    V2 a[U], b[U];
  };
  auto load = [&](Frag& f, int k0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int k = k0 + u * 4 + kq;  // neighbouring lane groups read neighbouring depths
      const bool in = k < K;
      const V2 x = pa[ka[in ? k : 0]], y = pb[kb[in ? k : 0]];
      f.a[u] = in ? x : V2{0, 0};
      f.b[u] = in ? y : V2{0, 0};
    }
  };
  ACC acc[3] = {ACC{0, 0, 0, 0}, ACC{0, 0, 0, 0}, ACC{0, 0, 0, 0}};
  auto products = [&](const Frag& f) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const V2 a = f.a[u], b = f.b[u];
      if constexpr (!G3) {
        acc[0] = mfma(a.x, b.x, acc[0]);
        acc[1] = mfma(a.x, b.y, acc[1]);
        acc[0] = mfma(-a.y, b.y, acc[0]);
        acc[1] = mfma(a.y, b.x, acc[1]);
      } else {
        acc[0] = mfma(a.x, b.x, acc[0]);
        acc[1] = mfma(a.y, b.y, acc[1]);
        acc[2] = mfma(a.x + a.y, b.x + b.y, acc[2]);
      }
    }
  };
  int k = wave * KS;
  Frag f0, f1;
  if (k < K) load(f0, k);
  while (k < K) {
    if (k + STEP < K) load(f1, k + STEP);
    products(f0);
    k += STEP;
    if (k >= K) break;
    if (k + STEP < K) load(f0, k + STEP);
    products(f1);
    k += STEP;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    V2 v;
    if constexpr (!G3)
      v = V2{acc[0][r], acc[1][r]};
    else
      v = V2{acc[0][r] - acc[1][r], acc[2][r] - acc[0][r] - acc[1][r]};
    red[wave][cpx<T>::row(kq, r) * 16 + r16] = v;
  }
  __syncthreads();
  for (int e = tid; e < 256; e += 64 * NW) {
    V2 s = red[0][e];
#pragma unroll
    for (int w = 1; w < NW; ++w) {
      s.x += red[w][e].x;
      s.y += red[w][e].y;
    }
    const int m = m0 + e / 16, n = n0 + e % 16;
    if (m >= M || n >= N) continue;
    T cr = p.are * s.x - p.aim * s.y, ci = p.are * s.y + p.aim * s.x;
    V2* c = p.C + p.cm.off(m) + p.cn.off(n);
    if (p.beta != T(0)) {
      const V2 y = *c;
      cr += p.beta * y.x;
      ci += p.beta * y.y;
    }
    *c = V2{cr, ci};
  }
}

// C = alpha sum_s P[s] + beta C for terms whose K was cut into p.K pieces;
// their partials, M x N each, follow one another at p.A.
template <typename T>
__global__ void __launch_bounds__(256) mreduce_kernel(MapGroup<T> g) {
  using V2 = typename cpx<T>::type;
  int ti = 0;
#pragma unroll
  for (int i = 1; i < kMapTerms; ++i)
    if (i < g.n && (int)blockIdx.x >= g.first[i]) ti = i;
  const MapTerm<T>& p = g.t[ti];
  const int mn = p.M * p.N, e = ((int)blockIdx.x - g.first[ti]) * 256 + (int)threadIdx.x;
  if (e >= mn) return;
  V2 s{0, 0};
#pragma unroll 4
  for (int q = 0; q < p.K; ++q) {
    const V2 x = p.A[(int64_t)q * mn + e];
    s.x += x.x;
    s.y += x.y;
  }
  T cr = p.are * s.x - p.aim * s.y, ci = p.are * s.y + p.aim * s.x;
  V2* c = p.C + p.cm.off(e / p.N) + p.cn.off(e % p.N);
  if (p.beta != T(0)) {
    const V2 y = *c;
    cr += p.beta * y.x;
    ci += p.beta * y.y;
  }
  *c = V2{cr, ci};
}

// A deep product of few tiles is cut along K into pieces of kMapPiece, summed
// by a second launch: a workgroup works off 1024 depths in 17 us (its CU's
// matrix cores, a 16 x 16 tile for 4 x 4 outputs), 256 in 7, and the sum takes
// 2.4.  Right product at o = 4, v = 16, FP64, two levels of that depth: 151 ->
// 138 us.  Beyond 32 tiles the products fill the launch by themselves.
constexpr int64_t kMapPiece = 256;
static int64_t map_pieces(const MappedProduct& p) {
  const int64_t tiles = ((p.m + 15) / 16) * ((p.n + 15) / 16);
  return p.k > 2 * kMapPiece && tiles <= 32 ? (p.k + kMapPiece - 1) / kMapPiece : 1;
}

template <typename T>
size_t mapped_gemm_workspace(const MappedProduct* p, int n) {
  int64_t e = 0;
  for (int i = 0; i < n; ++i)
    if (map_pieces(p[i]) > 1) e += map_pieces(p[i]) * p[i].m * p[i].n;
  return (size_t)e * 2 * sizeof(T);
}

template <typename T>
void launch_mapped_gemm(const MappedProduct* p, int n, void* ws, hipStream_t st) {
  using V2 = typename cpx<T>::type;
  auto side = [](int nd, const int64_t* dim, const int64_t* str) {
    const DevMap::Side d = DevMap::side(nd, dim, str);
    typename MapTerm<T>::Side s{};
    s.nd = nd;
    for (int k = 0; k < nd; ++k) {
      LRCC_REQUIRE(d.str[k] >= 0 && d.str[k] < INT32_MAX, LRCC_E_INTERNAL, "mapped product too large");
      s.dim[k] = d.dim[k], s.mul[k] = d.mul[k], s.sh[k] = (uint8_t)d.sh[k], s.str[k] = (int32_t)d.str[k];
    }
    return s;
  };
  MapGroup<T> g{}, red{};
  int64_t nb = 0, depth = 0, rb = 0;
  auto launch = [&] {
    if (g.n == 0) return;
    if (depth > 64 && nb < 512)
      hipLaunchKernelGGL((mgemm_kernel<T, 8>), dim3((unsigned)nb), dim3(64 * 8), 0, st, g);
    else
      hipLaunchKernelGGL((mgemm_kernel<T, 4>), dim3((unsigned)nb), dim3(64 * 4), 0, st, g);
    HIP_CHECK(hipGetLastError());
    g.n = 0, nb = 0, depth = 0;
  };
  auto reduce = [&] {  // after the products whose partials it sums
    if (red.n == 0) return;
    launch();
    hipLaunchKernelGGL(mreduce_kernel<T>, dim3((unsigned)rb), dim3(256), 0, st, red);
    HIP_CHECK(hipGetLastError());
    red.n = 0, rb = 0;
  };
  V2* part = (V2*)ws;
  for (int i = 0; i < n; ++i) {
    const MappedProduct& q = p[i];
    LRCC_REQUIRE(q.m > 0 && q.n > 0 && q.k > 0 && q.k <= kMapDepth && DevMap::fits(q.ma) && DevMap::fits(q.mb) &&
                     DevMap::fits(q.om) && q.ma.row(q.m - 1) + q.ma.col(q.k - 1) < INT32_MAX &&
                     q.mb.row(q.n - 1) + q.mb.col(q.k - 1) < INT32_MAX &&
                     q.om.row(q.m - 1) + q.om.col(q.n - 1) < INT32_MAX,
                 LRCC_E_INTERNAL, "mapped product too large");
    const int64_t nbm = (q.m + 15) / 16, tiles = nbm * ((q.n + 15) / 16);
    LRCC_REQUIRE(tiles < INT32_MAX / 2048, LRCC_E_INTERNAL, "mapped product too large");
    MapTerm<T> t{(const V2*)q.A,
                 (const V2*)q.B,
                 (V2*)q.C,
                 (T)q.are,
                 (T)q.aim,
                 (T)q.beta,
                 (int)q.m,
                 (int)q.n,
                 (int)q.k,
                 (int)nbm,
                 0,
                 side(q.ma.nm, q.ma.mdim, q.ma.mstr),
                 side(q.ma.nn, q.ma.ndim, q.ma.nstr),
                 side(q.mb.nm, q.mb.mdim, q.mb.mstr),
                 side(q.mb.nn, q.mb.ndim, q.mb.nstr),
                 side(q.om.nm, q.om.mdim, q.om.mstr),
                 side(q.om.nn, q.om.ndim, q.om.nstr)};
    const int64_t pieces = ws ? map_pieces(q) : 1;
    if (pieces > 1) {
      if (red.n == kMapTerms) reduce();
      MapTerm<T>& r = red.t[red.n];
      red.first[red.n++] = (int)rb;
      rb += (q.m * q.n + 255) / 256;
      r = t;
      r.A = part;
      r.K = (int)pieces;
      t.are = 1, t.aim = 0, t.beta = 0;
      const OutMap plain = OutMap::plain(q.n);
      t.cm = side(plain.nm, plain.mdim, plain.mstr), t.cn = side(plain.nn, plain.ndim, plain.nstr);
    }
    for (int64_t s = 0; s < pieces; ++s) {
      if (pieces > 1) {
        t.k0 = (int)(s * kMapPiece);
        t.K = (int)std::min(kMapPiece, q.k - s * kMapPiece);
        t.C = part;
        part += q.m * q.n;
      }
      if (g.n == kMapTerms) launch();
      g.t[g.n] = t;
      g.first[g.n++] = (int)nb;
      nb += tiles;
      depth = std::max<int64_t>(depth, t.K);
    }
  }
  launch();
  reduce();
}

// Variants: 0 and 1 share one 16 x 16 tile among 8 and 4 wavefronts, 2
// shares a 32 x 32 tile (8 wavefronts in FP64, 4 deeper-stepping ones in
// FP32: the FP64 accumulators leave registers for two-deep steps only), 3
// and 4 give every wavefront a 16 x 16 or a 16 x 32 tile of its own.
template <typename T>
void launch_wave_gemm(const WavePlan& p, bool ta, bool tb, int64_t m, int64_t n, int64_t k, double are, double aim,
                      const void* A, int64_t lda, const void* B, int64_t ldb, double bre, double bim, void* C,
                      const OutMap& om, int64_t cstride, hipStream_t st, bool conjb) {
  constexpr bool F64 = sizeof(T) == 8;
#define W_(TI, TJ, NW, KSP, U)                                                                                   \
  wgo<T, TI, TJ, NW, KSP, U>(ta, tb, m, n, k, are, aim, A, lda, B, ldb, bre, bim, C, om, st, p.splits, p.kchunk, \
                             cstride, conjb)
  switch (p.variant) {
    case 0: return W_(1, 1, 8, true, 4);
    case 1: return W_(1, 1, 4, true, 4);
    case 2: return W_(2, 2, F64 ? 8 : 4, true, F64 ? 2 : 4);
    case 3: return W_(1, 1, 4, false, 4);
    case 4: return W_(1, 2, 4, false, 4);
  }
#undef W_
  throw Error(LRCC_E_INTERNAL, "unknown wavefront GEMM variant");
}

// This kernel's time: as tiled_us, with the depth in place of slabs.  sigma is
// one depth of a layer of workgroups (variants 0 to 2: a 16 x 16 or 32 x 32 tile
// each; 3 and 4: four tiles), by transposition (A, B: NN, NT, TN, TT); delta is a
// depth's latency.  Fitted to the shapes of tiled_us that ran here; standard
// deviation FP64 4, 3, 6 % (variants 2, 3, 4), FP32 8, 6, 5 %.
namespace {
struct WaveCost {
  double call, f, reduce, tile, delta, sigma[4];
};
template <typename T>
double wave_us(const WavePlan& p, bool ta, bool tb, int64_t m, int64_t n) {
  static const WaveCost c64[3] = {{0.0, 0.07, 4.7, 4.4, 0.0026, {0.0326, 0.0332, 0.0323, 0.0327}},
                                  {2.8, 0.34, 4.0, 2.2, 0.0, {0.0051, 0.0051, 0.0113, 0.0130}},
                                  {3.0, 0.05, 4.0, 2.13, 0.0151, {0.0662, 0.0710, 0.0768, 0.0689}}};
  static const WaveCost c32[3] = {{1.0, 0.02, 4.3, 3.0, 0.0026, {0.0180, 0.0135, 0.0184, 0.0177}},
                                  {2.1, 0.20, 3.5, 0.96, 0.0331, {0.0134, 0.0101, 0.0186, 0.0157}},
                                  {2.6, 0.18, 2.0, 1.53, 0.0156, {0.0308, 0.0291, 0.0327, 0.0310}}};
  const WaveCost& c = (sizeof(T) == 8 ? c64 : c32)[p.variant - 2];
  const int64_t rows = p.variant == 2 ? 32 : 16, cols = p.variant == 3 ? 16 : 32, per = p.variant == 2 ? 1 : 4;
  const int64_t tiles = ((m + rows - 1) / rows) * ((n + cols - 1) / cols);
  const double layers = gemm_layers((tiles + per - 1) / per * p.splits, c.f);
  return c.call + layers * ((double)p.kchunk * c.sigma[ta * 2 + tb] + c.tile) + (double)p.kchunk * c.delta +
         (p.splits > 1 ? c.reduce : 0.0);
}
}  // namespace

// Which products run here, and how.  t16 and t32 count the 16 x 16 and
// 32 x 32 tiles of the output; figures are tiled kernel / this kernel in us.
//  * Addresses are 32-bit offsets from a tile's base: a leading dimension
//    beyond 2^32 bytes over 32 rows stays on the tiled kernel.
//  * Shallow (K <= 24): the output's traffic bounds both; the tiled kernel's
//    wider rows win from t16 = 8192 on (FP64 150x60000x20 79 / 94,
//    108000x10x10 (6750 tiles) 20 / 13).
//  * K <= 512 in FP64 on 1024 tiles or more: a tile per wavefront
//    (60000x150x150 274 / 252, 400x22500x400 581 / 542), except where the
//    64 x 64 tiles fit without padding (1200x14400x240 638 / 654: both
//    extents of 1000 or more).  FP32 is L2-bound there (44652x121x121
//    62 / 73) and takes the tiled kernel from 4096 tiles on.
//  * One 16 x 16 tile per workgroup where an extent is at most 16 or 32 x 32
//    tiles are few (FP64 600^3 42 against 48 on 32 x 32); 8 wavefronts below
//    512 tiles, 4 above.  These gain 1.2 times at least (but for one of 866 shapes).
//  * 32 x 32 tiles otherwise: in FP64 until 1024 tiles of 128 x 128 fill the
//    chip at the tiled kernel's higher intensity (18000x3000x3000 runs at 62-66
//    TFLOP/s there), in FP32 below 4e9 complex MACs or at most 96 wide
//    (1728x576x57600 2862 / 3511, 72x240x518400 999 / 810).
//  * Splits over K fill the chip's workgroup slots: at least 384 depths each
//    for the 16 x 16 tile, 256 for 32 x 32 (partials of at most 64 MB).
//  * A tile per wavefront and the 32 x 32 tiles only where their estimated time
//    is 3 % below the tiled kernel's.  The two are close once the chip is full,
//    and which one its last layer of tiles suits decides: FP64 NN 4000x3900x3000
//    6740 / 6135, NN 4000x3900x600 1381 / 1410, NT 9000x1700x3000 6225 / 6970, TN
//    9784x612x25 43 / 62; FP32 NN 388x4541x736 98 / 133, TT 1684x1374x1637 309 /
//    169.  Of 765 (FP64, 260 of them above 4e9 complex MACs) and 517 (FP32)
//    shapes run here without this line, 67 and 36 lost 3 % or more, up to 45 %;
//    with it one and none, and the mean gain over all shapes is no less (2.733
//    -> 2.740 and 2.562 -> 2.567 times, large FP64 ones 1.076 -> 1.075).
template <typename T>
WavePlan wave_plan(bool ta, bool tb, int64_t m, int64_t n, int64_t k, int64_t lda, int64_t ldb, bool can_split) {
  constexpr bool F64 = sizeof(T) == 8;
  WavePlan p;
  if (m <= 0 || n <= 0 || k <= 0) return p;
  if (std::max(lda, ldb) * 32 * (int64_t)(2 * sizeof(T)) >= (int64_t(1) << 32)) return p;
  auto cdiv = [](int64_t a, int64_t b) { return (a + b - 1) / b; };
  const int64_t t16 = cdiv(m, 16) * cdiv(n, 16), t32 = cdiv(m, 32) * cdiv(n, 32);
  const bool narrow = std::min(m, n) <= 16;
  int64_t slots = 0, mink = 0, tiles = 0;
  if (k <= 24) {
    if (t16 >= 8192) return p;
    p.variant = t16 >= 1024 ? 3 : 1;
  } else if (k <= 512 && t16 >= 1024) {
    if (F64 ? std::min(m, n) >= 1000 : t16 >= 4096) return p;
    p.variant = narrow ? 3 : 4;
  } else if (narrow || (k < 2048 && t32 < (F64 ? 900 : 256))) {
    p.variant = t16 < 512 ? 0 : 1;
    slots = 512, mink = 384, tiles = t16;
  } else {
    if (F64 ? cdiv(m, 128) * cdiv(n, 128) >= 1024 : ((double)m * n * k >= 4e9 && std::min(m, n) > 96)) return p;
    p.variant = 2;
    slots = F64 ? 256 : 512, mink = 256, tiles = t32;
  }
  p.kchunk = k;
  if (can_split && tiles > 0 && tiles < 2 * slots) {
    const int64_t part = m * n * (int64_t)(2 * sizeof(T));
    const int64_t smax = std::min<int64_t>({64, k / mink, (int64_t(64) << 20) / part});
    auto eff = [&](int64_t s) {
      const int64_t w = tiles * s, rounds = cdiv(w, slots);
      return (double)w / (double)(rounds * slots);
    };
    double best = 0;
    for (int64_t s = 1; s <= smax; ++s) best = std::max(best, eff(s));
    for (int64_t s = 1; s <= smax; ++s)
      if (eff(s) >= 0.9 * best) {
        if (s > 1 && eff(s) >= 1.15 * eff(1)) {
          p.kchunk = cdiv(cdiv(k, s), 16) * 16;
          p.splits = (int)cdiv(k, p.kchunk);
        }
        break;
      }
  }
  if (p.variant >= 2) p.us = wave_us<T>(p, ta, tb, m, n);
  if (p.us >= 0.97 * tiled_us(F64, ta, tb, m, n, k, can_split)) return WavePlan();
  return p;
}

#define INST_(T)                                                                                                    \
  template void launch_wave_gemm<T>(const WavePlan&, bool, bool, int64_t, int64_t, int64_t, double, double,         \
                                    const void*, int64_t, const void*, int64_t, double, double, void*,              \
                                    const OutMap&, int64_t, hipStream_t, bool);                                     \
  template WavePlan wave_plan<T>(bool, bool, int64_t, int64_t, int64_t, int64_t, int64_t, bool);                    \
  template size_t mapped_gemm_workspace<T>(const MappedProduct*, int);                                              \
  template void launch_mapped_gemm<T>(const MappedProduct*, int, void*, hipStream_t);
INST_(double)
INST_(float)
#undef INST_

}  // namespace lrcc
