// Complex FP32 GEMM on the BF16 matrix cores, for large products.
//
// The FP32 MFMA rate bounds the tiled kernel (119 TFLOP/s of 157 in the 3M
// count); BF16 runs at 16 times that rate.  An FP32 number is exactly the
// sum of three BF16 numbers, x = h + m + l (8 significant bits each,
// round to nearest; G. Henry, P. T. P. Tang and A. Heinecke, ARITH 2019), so a
// real FP32 product is six BF16 products,
//   x y = h h + h m + m h + m m + h l + l h,
// each exact in FP32 and added up in FP32 by the MFMA: 18 BF16 products for
// one complex 3M product, 2.7 times fewer matrix-core cycles than the FP32
// instruction needs.  m l + l m + l l, left out, is below 2^-24 |x y| (|m| <=
// 2^-8, |l| <= 2^-17 of x's binade; 2^-27.5 in the mean).
//
// split_pack_kernel writes both operands as the LDS image the product reads:
// blocks of 128 rows x 16 depths, for each of re, im and re + im (the 3M
// sums, rounded to FP32 as in the tiled kernel) and each of h, m, l, eight
// consecutive depths of a row in 16 bytes.  Transposes, conjugation and
// padding end there (zeros beyond the operand), so one product kernel serves
// all layouts and its loads go straight from global memory to LDS.
//
// split_gemm_kernel: a 256 x 128 tile on 8 wavefronts of 64 x 64 (or 128 x
// 128 on 4), two LDS stages, the next one in flight during the products.
// P1 = Ar Br, P2 = Ai Bi and P3 = (Ar+Ai)(Br+Bi) are accumulated one after
// the other over the whole depth, P3 on top of -P1 - P2, so 128 accumulator
// registers hold a 64 x 64 complex tile and leave room for the fragments at
// two wavefronts per SIMD; a 3M tile with all three at once would not fit.
//
// What bounds it: power.  In the large launches of a right product (o = 20, v =
// 150, 24 vectors) the matrix cores are busy 57-63 % of the cycles, at 1.85 GHz of
// 2.4; short launches run at 2.1-2.3 GHz.  A register-only BF16 MFMA loop on
// normal data sustains 1.3-1.5 PFLOP/s of the nominal 2.5 on this card, the kernel
// 1.1-1.2.  HBM traffic is 0.9 TB/s, LDS bank conflicts nil.  Measured, TFLOP/s in the 6 MNK count, tiled -> this (packing
// apart): 18000x3000x3000 121 -> 196, 4560x11175x11175 118 -> 190,
// 2280x11175x3000 111 -> 185.
//
// Accuracy: the MFMA adds 16 products before it rounds into the accumulator,
// where the FP32 instruction adds 4, so the error against 64 bits is smaller
// at equal depth (18000x3000x3000 1.19e-6 against 1.39e-6 in the 2-norm).
// kChain bounds the depth of one accumulation chain, so that it stays below
// that of the tiled kernel where that one splits K, too.
//
// Range: BF16 has FP32's exponents but not its significand's reach below
// them, so the operands are packed 2^24 times larger.  FP32 numbers, the
// subnormal ones among them, are multiples of 2^-149; scaled, h, m and l are
// multiples of 2^-125, normal BF16 numbers or zero, and the split is exact.
// Below 2^32 in magnitude the scaled values (2^56), their 3M sums (2^57) and
// the sum of kChain products (2^126) stay finite.  An element of 2^32 or
// more, an infinity or a NaN in either operand sets a flag, and that product
// runs on the FP32 MFMA instead: the flag is read on the device, by the
// product kernel, which then returns at once, and by a tiled launch behind it
// (launch_gemm_if), which otherwise does.  The packing's check is hidden
// behind its memory traffic; the launches that do nothing cost 0.4 % of a right
// product (o = 20, v = 150, 24 vectors: 91.4 -> 91.8 ms); a product that the flag
// sends to the FP32 MFMA takes 7 % more time than without the packing (mean of
// 120 products of 2e9 to 3e10 complex MACs).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma.h"

namespace lrcc {

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef float f16v __attribute__((ext_vector_type(16)));

namespace {
constexpr int kRB = 128;                       // rows of a packed block
constexpr int kSlab = 16;                      // depths of a packed slab
constexpr int kChunk = kRB * kSlab * 3 * 2;    // bytes of one block x slab x component (three BF16 terms)

constexpr float kScale = 0x1p24f, kUnscale = 0x1p-48f;  // of an operand, of a product
constexpr float kLargest = 0x1p32f;                     // magnitudes from here on take the FP32 MFMA
constexpr size_t kFlagBytes = 256;

__device__ inline uint16_t bits(__bf16 x) { return __builtin_bit_cast(uint16_t, x); }

// x = h + m + l exactly, for x a multiple of 2^-125 below 2^58
__device__ inline void split3(float x, uint16_t& h, uint16_t& m, uint16_t& l) {
  const __bf16 bh = (__bf16)x;
  const float r = x - (float)bh;
  const __bf16 bm = (__bf16)r;
  h = bits(bh);
  m = bits(bm);
  l = bits((__bf16)(r - (float)bm));
}
}  // namespace

// One workgroup: 128 rows x 16 depths at a time, read along the operand's
// contiguous dimension (rows with KMAJ, else depths) and turned in LDS, so that
// every thread splits eight consecutive depths of one row and writes 16 bytes
// per component and term.  With MAP the element (r, k) lies at X + map.row(r0
// + r) + map.col(k0 + k).  *flag is set where an element is out of range.  Bound
// by memory: 8 bytes read and 18 written per element.
template <bool KMAJ, bool MAP>
__global__ void __launch_bounds__(256)
    split_pack_kernel(int64_t rows, int64_t K, const float2* __restrict__ X, int64_t ld, DevMap map, int64_t rbase,
                      int64_t kbase, float sgn, int64_t nslab, uint4* __restrict__ P, int* __restrict__ flag) {
  __shared__ float2 t[kRB][kSlab + 1];
  bool bad = false;
  constexpr int NQ = kRB * kSlab / 256;
  const int tid = threadIdx.x;
  const int64_t r0 = (int64_t)blockIdx.x * kRB;
  int64_t roff[KMAJ ? 1 : NQ];
  if constexpr (MAP) {
#pragma unroll
    for (int q = 0; q < (KMAJ ? 1 : NQ); ++q) {
      const int64_t r = r0 + (KMAJ ? tid % kRB : (q * 256 + tid) / kSlab);
      roff[q] = map.row(rbase + (r < rows ? r : 0));
    }
  }
  for (int64_t s = blockIdx.y; s < nslab; s += gridDim.y) {
    const int64_t k0 = s * kSlab;
    int64_t koff = 0;
    if constexpr (MAP && !KMAJ) {
      const int64_t k = k0 + tid % kSlab;
      koff = map.col(kbase + (k < K ? k : 0));
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const int e = q * 256 + tid;
      const int row = KMAJ ? e % kRB : e / kSlab, kk = KMAJ ? e / kRB : e % kSlab;
      const int64_t r = r0 + row, k = k0 + kk;
      const bool in = r < rows && k < K;
      int64_t at;
      if constexpr (!MAP)
        at = KMAJ ? k * ld + r : r * ld + k;
      else if constexpr (KMAJ)
        at = roff[0] + map.col(kbase + (k < K ? k : 0));
      else
        at = roff[q] + koff;
      const float2 v = X[MAP || in ? at : 0];
      bad |= in && !(__builtin_fabsf(v.x) < kLargest && __builtin_fabsf(v.y) < kLargest);
      t[row][kk] = in ? float2{v.x * kScale, v.y * (sgn * kScale)} : float2{0.0f, 0.0f};
    }
    __syncthreads();
    const int row = tid & (kRB - 1), kg = tid >> 7;
    float2 x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = t[row][kg * 8 + e];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      uint32_t w[3][4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        uint16_t u[2][3];
#pragma unroll
        for (int z = 0; z < 2; ++z) {
          const float2 v = x[2 * q + z];
          split3(c == 0 ? v.x : c == 1 ? v.y : v.x + v.y, u[z][0], u[z][1], u[z][2]);
        }
#pragma unroll
        for (int p = 0; p < 3; ++p) w[p][q] = (uint32_t)u[0][p] | ((uint32_t)u[1][p] << 16);
      }
      uint4* d = P + (((int64_t)blockIdx.x * 3 + c) * nslab + s) * (kChunk / 16);
#pragma unroll
      for (int p = 0; p < 3; ++p) d[(p * 2 + kg) * kRB + row] = uint4{w[p][0], w[p][1], w[p][2], w[p][3]};
    }
    __syncthreads();
  }
  if (bad) *flag = 1;
}

__global__ void split_clear_kernel(int* flags) { flags[threadIdx.x] = 0; }

// A mapped operand as [row][k], for the FP32 MFMA: where a flag is set.
__global__ void __launch_bounds__(256) split_copy_kernel(const int* __restrict__ flags, int64_t rows, int64_t K,
                                                         const float2* __restrict__ X, DevMap map, int64_t rbase,
                                                         int64_t kbase, float2* __restrict__ out) {
  if (!(flags[0] | flags[1])) return;
  for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < rows * K; e += (int64_t)gridDim.x * 256)
    out[e] = X[map.row(rbase + e / K) + map.col(kbase + e % K)];
}

template <int WGM, int WGN, int NS>  // NS slabs per stage
__global__ void __launch_bounds__(64 * WGM * WGN, 2)
    split_gemm_kernel(int64_t M, int64_t N, int64_t nslab, const char* __restrict__ Ap, const char* __restrict__ Bp,
                      float are, float aim, float bre, float bim, float2* __restrict__ C, DevMap om, int64_t om0,
                      int64_t on0, int64_t schunk, int64_t cstride, const int* __restrict__ flags) {
  if (flags[0] | flags[1]) return;
  constexpr int NW = WGM * WGN, BM = 64 * WGM, BN = 64 * WGN;
  constexpr int RA = BM / kRB, RB = BN / kRB;
  constexpr int STAGE = (RA + RB) * NS * kChunk;
  __shared__ __align__(16) char lds[2][STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, kg = lane >> 5;
  const int wm = (wave / WGN) * 64, wn = (wave % WGN) * 64;
  const int64_t nbm = (M + BM - 1) / BM, nbn = (N + BN - 1) / BN;
  int64_t tm, tn;
  tile_of(blockIdx.x, nbm, nbn, tm, tn);
  const int64_t s0 = (int64_t)blockIdx.y * schunk;
  const int64_t ns = (nslab < s0 + schunk ? nslab : s0 + schunk) - s0;
  C += (int64_t)blockIdx.y * cstride;
  const int64_t nrbA = (M + kRB - 1) / kRB, nrbB = (N + kRB - 1) / kRB;

  // Stage t of component c: NS consecutive slabs of every row block, copied
  // as they lie (1 KB per wavefront load).  Blocks beyond the operand feed
  // outputs that are never stored; they read its last block.
  constexpr int PER = NS * kChunk / 1024, TOT = (RA + RB) * PER, NQ = TOT / NW;
  static_assert(TOT % NW == 0, "stage does not split over the wavefronts");
  const char* src[NQ];
  int dst[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    const int x = q * NW + wave, b = x / PER, o = x % PER;
    const bool isa = b < RA;
    const int64_t blk = isa ? tm * RA + b : tn * RB + (b - RA), last = (isa ? nrbA : nrbB) - 1;
    const uintptr_t base = isa ? (uintptr_t)Ap : (uintptr_t)Bp;
    src[q] = (const char*)(base + ((blk < last ? blk : last) * 3 * nslab + s0) * kChunk + o * 1024);
    dst[q] = b * NS * kChunk + o * 1024;
  }
  auto issue = [&](int buf, int c, int64_t t) __attribute__((always_inline)) {
    const int64_t at = (c * nslab + t * NS) * kChunk;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
      __builtin_amdgcn_global_load_lds(
          (const __attribute__((address_space(1))) void*)(src[q] + at + lane * 16),
          (__attribute__((address_space(3))) void*)(lds[buf] + dst[q]), 16, 0, 0);
  };
  f16v acc[2][2][2];
#pragma unroll
  for (int p = 0; p < 2; ++p)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[p][i][j] = f16v{0};
  const int ra = (wm / kRB) * NS * kChunk + (kg * kRB + wm % kRB + l32) * 16;
  const int rb = (RA + wn / kRB) * NS * kChunk + (kg * kRB + wn % kRB + l32) * 16;
  auto compute = [&](int buf, f16v(&a)[2][2]) __attribute__((always_inline)) {
    const char* L = lds[buf];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      bf8 fa[3][2], fb[3][2];
#pragma unroll
      for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          fa[p][i] = *(const bf8*)(L + ra + s * kChunk + p * (kChunk / 3) + i * 512);
          fb[p][i] = *(const bf8*)(L + rb + s * kChunk + p * (kChunk / 3) + i * 512);
        }
      // small terms first; m l, l m and l l lie below FP32's rounding
      constexpr int PA[6] = {0, 2, 1, 0, 1, 0}, PB[6] = {2, 0, 1, 1, 0, 0};
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j)
            a[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[PA[t]][i], fb[PB[t]][j], a[i][j], 0, 0, 0);
    }
  };
  const int64_t nt = (ns + NS - 1) / NS;
  int buf = 0;
  issue(0, 0, 0);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  auto pass = [&](int c, f16v(&a)[2][2]) __attribute__((always_inline)) {
    for (int64_t t = 0; t < nt; ++t) {
      if (t + 1 < nt)
        issue(buf ^ 1, c, t + 1);
      else if (c < 2)
        issue(buf ^ 1, c + 1, 0);
      compute(buf, a);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      buf ^= 1;
    }
  };
  pass(0, acc[0]);
  pass(1, acc[1]);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const f16v p1 = acc[0][i][j], p2 = acc[1][i][j];
      acc[0][i][j] = p1 - p2;
      acc[1][i][j] = -p1 - p2;
    }
  pass(2, acc[1]);

  const bool use_beta = (bre != 0.0f || bim != 0.0f);
  int64_t coff[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int64_t n = tn * BN + wn + j * 32 + l32;
    coff[j] = n < N ? om.col(on0 + n) : -1;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int64_t m = tm * BM + wm + i * 32 + (r / 4) * 8 + kg * 4 + r % 4;
      if (m >= M) continue;
      const int64_t roff = om.row(om0 + m);
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        if (coff[j] < 0) continue;
        const float re = acc[0][i][j][r] * kUnscale, im = acc[1][i][j][r] * kUnscale;
        float cr = are * re - aim * im, ci = are * im + aim * re;
        float2* c = C + roff + coff[j];
        if (use_beta) {
          const float2 y = *c;
          cr += bre * y.x - bim * y.y;
          ci += bre * y.y + bim * y.x;
        }
        *c = float2{cr, ci};
      }
    }
}

namespace {
constexpr int64_t kChain = 3072;                    // deepest accumulation chain
int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }
int64_t slabs(int64_t k) { return cdiv(k, 2 * kSlab) * 2; }  // padded to whole stages
size_t pack_bytes(int64_t rows, int64_t k) { return (size_t)(cdiv(rows, kRB) * 3 * slabs(k)) * kChunk; }

void pack(bool kmaj, int64_t rows, int64_t k, const void* X, int64_t ld, bool conj, void* P, int* flag,
          hipStream_t st, const OutMap* map = nullptr, int64_t r0 = 0, int64_t k0 = 0) {
  const int64_t ns = slabs(k);
  const dim3 grid((unsigned)cdiv(rows, kRB), (unsigned)std::min<int64_t>(ns, 4096));
  if (map) kmaj = map->mstr[map->nm - 1] == 1;
  const DevMap dm(map ? *map : OutMap::plain(ld));
#define PACK_(KM, MP)                                                                                              \
  hipLaunchKernelGGL((split_pack_kernel<KM, MP>), grid, dim3(256), 0, st, rows, k, (const float2*)X, ld, dm, r0, k0, \
                     conj ? -1.0f : 1.0f, ns, (uint4*)P, flag)
  if (kmaj && map)
    PACK_(true, true);
  else if (kmaj)
    PACK_(true, false);
  else if (map)
    PACK_(false, true);
  else
    PACK_(false, false);
#undef PACK_
  HIP_CHECK(hipGetLastError());
}
}  // namespace

// This kernel's time with the plan p, as tiled_us: layers of workgroups, one per
// CU of the 256 x 128 tile, sigma a depth and `tile` a tile for its fill, drain
// and output; two of the 128 x 128 tile share a CU, so that a layer of half the
// work overlaps the next one but for delta a depth.  Packing, output and partials
// are traffic, in us per million elements.  Fitted to 308 products of 2e9 to 3e10
// complex MACs, in one and in several blocks; standard deviation 4 % (6 % with
// the smaller tile).  Those are over before the card's power limit tells: a
// longer run comes to 195 TFLOP/s (180 with the smaller tile) on the padded
// extents, which leaves 18000x3000x3000 at 5150 us (measured 4960) and
// 540000x400x400 at 5030 (4610), packing included.
namespace {
double split_us(const SplitPlan& p, int64_t m, int64_t n, int64_t k) {
  const double sigma = p.small ? 0.090 : 0.1815, delta = p.small ? 0.065 : 0.0, f = p.small ? 0.68 : 0.0,
               tile = p.small ? 2.4 : 12.2, call = 5.0, packing = 6.5e-6, out = 1.2e-6, part = 1.8e-6;
  const double sustained = 6.0 / (p.small ? 180e6 : 195e6);
  const int64_t bm = p.small ? 128 : 256, nm = cdiv(m, p.mc), nn = cdiv(n, p.nc), nk = cdiv(k, p.kl);
  double us = packing * (double)k * ((double)n + (double)m * (double)(nm > 1 ? nn : 1));
  for (int e = 0; e < 8; ++e) {  // the full and the last block of rows, of columns, of depth
    const int64_t cm = e & 1 ? 1 : nm - 1, cn = e & 2 ? 1 : nn - 1, ck = e & 4 ? 1 : nk - 1;
    const int64_t mb = e & 1 ? m - (nm - 1) * p.mc : p.mc, nb = e & 2 ? n - (nn - 1) * p.nc : p.nc,
                  kb = e & 4 ? k - (nk - 1) * p.kl : p.kl;
    if (cm * cn * ck == 0) continue;
    const double tiles = (double)(cdiv(mb, bm) * cdiv(nb, 128)), mn = (double)mb * (double)nb;
    const double depth = (double)kb / p.splits;
    const double layers = gemm_layers((int64_t)tiles * p.splits, f) * (depth * sigma + tile) + depth * delta;
    const double power = sustained * tiles * (double)(bm * 128) * (double)kb;
    us += (double)(cm * cn * ck) *
          (call + std::max(layers, power) + out * mn + (p.splits > 1 ? part * mn * p.splits : 0.0));
  }
  return us;
}
}  // namespace

// The plan of least estimated time that fits the budget: chains of K side by side
// into partials, depth of a pass, row blocks of either operand, with the smaller
// tile where the larger one pads the rows by 7 % more.  It is taken where it saves 5 % of the FP32 kernels' estimate.  Row blocks leave a
// launch few tiles, shorter passes read and write the output once more: 9814 x
// 374 x 3986 in 256 MiB, rows of one operand in five blocks, took 1976 us
// (tiled 959).  Below a depth of 256 the output's traffic is no longer hidden,
// one workgroup per CU (480x450000x150 2460 -> 2670); below 2e9 MACs the
// wavefront kernel or the launches decide.  Measured, FP32 MFMA -> here, us:
// 540000x400x400 5330 -> 4610, 8052x671x671 224 -> 205.
SplitPlan split_plan(bool ta, bool tb, int64_t m, int64_t n, int64_t k, size_t budget) {
  SplitPlan best;
  if (m <= 0 || n <= 0 || k < 256 || (double)m * n * k < 2e9) return best;
  const WavePlan w = wave_plan<float>(ta, tb, m, n, k, ta ? m : k, tb ? k : n, true);
  if (w.variant == 0 || w.variant == 1) return best;  // an extent of at most 16
  double least = 0.95 * (w.variant > 0 ? w.us : tiled_us(false, ta, tb, m, n, k, true));
  auto consider = [&](const SplitPlan& q) {
    const double us = split_us(q, m, n, k);
    if (us >= least) return;
    least = us;
    best = q;
    best.use = true;
  };
  const int64_t lesser = std::min(m, n), larger = std::max(m, n);
  const bool small_tile = 195.0 * (double)cdiv(m, 128) < 180.0 * 2.0 * (double)cdiv(m, 256);
  for (int64_t s = 1; s <= std::min<int64_t>(8, std::max<int64_t>(1, k / 512)); ++s)
    for (int64_t c0 = cdiv(k, kChain * s), c = c0; c < c0 + 4; ++c) {  // c passes of s chains each
      const int64_t chain = cdiv(cdiv(k, c * s), 2 * kSlab) * 2 * kSlab;
      if (c > c0 && chain < 512) break;
      SplitPlan q;
      q.small = small_tile;
      q.splits = (int)s;
      q.kl = std::min(k, chain * s);
      const size_t block = pack_bytes(kRB, q.kl), part = s > 1 ? (size_t)s * 8 : 0;
      for (int64_t parts = 1; parts <= 16; ++parts) {
        // blocks of the lesser extent, and the largest of the other one beside them
        const int64_t lb = parts == 1 ? lesser : cdiv(cdiv(lesser, parts), 256) * 256;
        const size_t held = pack_bytes(lb, q.kl) + kFlagBytes;
        int64_t gb = held < budget ? (int64_t)((budget - held) / (block + part * lb * kRB)) * kRB : 0;
        if (gb >= larger)
          gb = larger;
        else if (gb < 256)
          continue;
        else
          gb = cdiv(cdiv(larger, cdiv(larger, gb / 256 * 256)), 256) * 256;
        q.mc = m >= n ? gb : lb, q.nc = m >= n ? lb : gb;
        q.a_bytes = pack_bytes(q.mc, q.kl);
        q.b_bytes = pack_bytes(q.nc, q.kl);
        q.bytes = q.a_bytes + q.b_bytes + part * q.mc * q.nc + kFlagBytes;
        if (q.bytes <= budget) consider(q);
        if (gb == larger) break;  // smaller blocks only cost more
      }
      if (q.mc == m && q.nc == n) break;  // and so do shorter passes
    }
  return best;
}

void launch_split_gemm(const SplitPlan& p, bool ta, bool tb, int64_t m, int64_t n, int64_t k, double are, double aim,
                       const void* A, int64_t lda, const void* B, int64_t ldb, double bre, double bim, void* C,
                       const OutMap& om, void* ws, hipStream_t st, bool conjb) {
  LRCC_REQUIRE((!p.amap || DevMap::fits(p.ma)) && (!p.bmap || DevMap::fits(p.mb)), LRCC_E_INTERNAL,
               "operand map: more than 2^31 rows or depths");
  char* Pa = (char*)ws;
  char* Pb = Pa + p.a_bytes;
  char* part = Pb + p.b_bytes;
  // Set in one block of the product, a flag holds for the later ones, too.
  int* flags = (int*)((char*)ws + p.bytes - kFlagBytes);
  hipLaunchKernelGGL(split_clear_kernel, dim3(1), dim3(2), 0, st, flags);
  HIP_CHECK(hipGetLastError());
  auto copy = [&](int64_t rows, int64_t kl, const void* X, const OutMap& map, int64_t r0, int64_t k0, void* out) {
    const unsigned blocks = (unsigned)std::min<int64_t>(cdiv(rows * kl, 256), 4096);
    hipLaunchKernelGGL(split_copy_kernel, dim3(blocks), dim3(256), 0, st, flags, rows, kl, (const float2*)X,
                       DevMap(map), r0, k0, (float2*)out);
    HIP_CHECK(hipGetLastError());
  };
  const int64_t bm = p.small ? 128 : 256;
  for (int64_t k0 = 0; k0 < k; k0 += p.kl) {
    const int64_t kl = std::min(p.kl, k - k0), ns = slabs(kl);
    const int64_t sc = cdiv(cdiv(ns, p.splits), 2) * 2;
    const int splits = (int)cdiv(ns, sc);
    const double br = k0 == 0 ? bre : 1.0, bi = k0 == 0 ? bim : 0.0;
    bool a_packed = false;
    for (int64_t n0 = 0; n0 < n; n0 += p.nc) {
      const int64_t nc = std::min(p.nc, n - n0);
      const char* Bx = (const char*)B + (tb ? n0 * ldb + k0 : k0 * ldb + n0) * 8;
      if (p.bmap)
        pack(false, nc, kl, B, 0, conjb, Pb, flags + 1, st, &p.mb, n0, k0);
      else
        pack(!tb, nc, kl, Bx, ldb, conjb, Pb, flags + 1, st);
      for (int64_t m0 = 0; m0 < m; m0 += p.mc) {
        const int64_t mc = std::min(p.mc, m - m0);
        const char* Ax = (const char*)A + (ta ? k0 * lda + m0 : m0 * lda + k0) * 8;
        if ((!a_packed || p.mc < m) && p.amap)
          pack(false, mc, kl, A, 0, false, Pa, flags, st, &p.ma, m0, k0);
        else if (!a_packed || p.mc < m)
          pack(ta, mc, kl, Ax, lda, false, Pa, flags, st);
        a_packed = true;
        const int64_t nb = cdiv(mc, bm) * cdiv(nc, 128);
        LRCC_REQUIRE(nb < (int64_t(1) << 31), LRCC_E_INVALID, "gemm grid too large");
        const dim3 grid((unsigned)nb, (unsigned)splits);
        const bool parts = splits > 1;
        const OutMap mo = parts ? OutMap::plain(nc) : om;
        const float al[2] = {parts ? 1.0f : (float)are, parts ? 0.0f : (float)aim};
        const float be[2] = {parts ? 0.0f : (float)br, parts ? 0.0f : (float)bi};
        float2* out = (float2*)(parts ? part : (char*)C);
        const int64_t om0 = parts ? 0 : m0, on0 = parts ? 0 : n0;
        if (p.small)
          hipLaunchKernelGGL((split_gemm_kernel<2, 2, 1>), grid, dim3(256), 0, st, mc, nc, ns, Pa, Pb, al[0], al[1],
                             be[0], be[1], out, DevMap(mo), om0, on0, sc, mc * nc, flags);
        else
          hipLaunchKernelGGL((split_gemm_kernel<4, 2, 2>), grid, dim3(512), 0, st, mc, nc, ns, Pa, Pb, al[0], al[1],
                             be[0], be[1], out, DevMap(mo), om0, on0, sc, mc * nc, flags);
        HIP_CHECK(hipGetLastError());
        if (p.amap) copy(mc, kl, A, p.ma, m0, k0, Pa);
        if (p.bmap) copy(nc, kl, B, p.mb, n0, k0, Pb);
        launch_gemm_if(flags, ta && !p.amap, tb || p.bmap, mc, nc, kl, al[0], al[1], p.amap ? Pa : Ax,
                       p.amap ? kl : lda, p.bmap ? Pb : Bx, p.bmap ? kl : ldb, be[0], be[1], out, mo, om0, on0, splits,
                       sc * kSlab, conjb, st);
        if (parts) launch_splitk_reduce_f32(mc, nc, splits, part, are, aim, br, bi, C, om, m0, n0, st);
      }
    }
  }
}

}  // namespace lrcc
