// The splits of dw_o's contraction over the tokens: the ranges that launch_gemm_tn makes of them
// (whole 32-index stages) are never more than the partials that the workspace holds, and the
// count does not jump between a token count and the next (it did where one was a multiple of
// 32), up to 4096 tokens.
#include <stdio.h>

#include "gemm_plan.hpp"

using namespace laga;

int main() {
  long long split = 0, bad = 0;
  for (int F = 16; F <= 16384; F += F < 512 ? 48 : 1008)
    for (int D = 16; D <= 7168; D += D < 512 ? 48 : 1008)
      for (int T = 1; T < 20000; T += T < 1200 ? 1 : 487)
        for (int esize = 2; esize <= 4; esize += 2) {
          const int n = gemm_tn_splits(F, D, T, esize), chunk = ((T + n - 1) / n + 31) / 32 * 32;
          const int ranges = (T + chunk - 1) / chunk, next = gemm_tn_splits(F, D, T + 1, esize);
          split += n > 1;
          if (n < 1 || ranges > n || (T + 1 < 4096 && (next < n || next > n + 1)))
            if (bad++ < 5) printf("F %d D %d T %d: %d splits (%d at T + 1), %d ranges\n", F, D, T, n, next, ranges);
        }
  printf("%lld split contractions, %lld wrong\n", split, bad);
  return bad != 0 || split == 0;
}
