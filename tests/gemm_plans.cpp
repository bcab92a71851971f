// Prints the library's GEMM plans for the products on stdin (test_gemm_plans.py).
//   w fp64 ta tb m n k         wavefront kernel: variant and splits with and without workspace
//   s ta tb m n k budget       BF16 kernel: use, splits, block rows, columns and depth, bytes
//   y                          memory given back to a failing allocation: 1 if as promised
#include <cstdio>

#include "common.h"
#include "devmem.h"
#include "kernels.h"

using namespace lrcc;

// An arena of 1 MiB (bookkeeping only, never dereferenced), 600 KB of it held by
// something that yields.
static bool yields() {
  Arena a(reinterpret_cast<void*>(uintptr_t(1) << 32), 1 << 20);
  ArenaScope in(&a);
  struct Holder : Yields {
    void* p = dev_alloc(600 << 10);
    int asked = 0;
    bool yield() override {
      ++asked;
      if (!p) return false;
      dev_free(p);
      p = nullptr;
      return true;
    }
  } h;
  auto fails = [](size_t b) {
    try {
      dev_alloc(b);
      return false;
    } catch (const Error& e) {
      return e.code == LRCC_E_NOMEM;
    }
  };
  if (!fails(700 << 10)) return false;  // no scope: nobody is asked
  YieldScope scope(&h);
  {
    YieldScope none(nullptr);
    if (!fails(700 << 10) || h.asked != 0) return false;
  }
  dev_alloc(100 << 10);  // fits
  if (h.asked != 0) return false;
  dev_alloc(550 << 10);  // fits in what is given back
  if (h.asked != 1 || h.p) return false;
  return fails(500 << 10) && h.asked == 2;  // nothing left to give
}

int main() {
  char what;
  while (scanf(" %c", &what) == 1) {
    if (what == 'w') {
      int f, ta, tb;
      long m, n, k;
      if (scanf("%d %d %d %ld %ld %ld", &f, &ta, &tb, &m, &n, &k) != 6) return 1;
      const long lda = ta ? m : k, ldb = tb ? k : n;
      for (int ws = 1; ws >= 0; --ws) {
        const WavePlan p = f ? wave_plan<double>(ta, tb, m, n, k, lda, ldb, ws)
                             : wave_plan<float>(ta, tb, m, n, k, lda, ldb, ws);
        printf("%d %d ", p.variant, p.splits);
      }
      printf("\n");
    } else if (what == 's') {
      int ta, tb;
      long m, n, k, budget;
      if (scanf("%d %d %ld %ld %ld %ld", &ta, &tb, &m, &n, &k, &budget) != 6) return 1;
      const SplitPlan p = split_plan(ta, tb, m, n, k, (size_t)budget);
      printf("%d %d %ld %ld %ld %ld\n", p.use, p.splits, (long)p.mc, (long)p.nc, (long)p.kl, (long)p.bytes);
    } else if (what == 'y') {
      printf("%d\n", yields());
    } else {
      return 1;
    }
  }
  return 0;
}
