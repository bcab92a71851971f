// Prints the library's GEMM plans for the products on stdin (test_gemm_plans.py).
//   w fp64 ta tb m n k         wavefront kernel: variant and splits with and without workspace
//   s ta tb m n k budget       BF16 kernel: use, splits, block rows, columns and depth, bytes
#include <cstdio>

#include "common.h"
#include "kernels.h"

int main() {
  using namespace lrcc;
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
    } else {
      return 1;
    }
  }
  return 0;
}
