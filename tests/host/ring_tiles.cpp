// The bf16 GEMM's tile shape over the sizes of its output: the middle one is launched only where
// it gives enough workgroups and fits the CUs at once (a second round of a few workgroups loses
// to large tiles in one), the small one only where neither other shape gives enough.
#include <stdio.h>

#include "gemm_plan.hpp"

using namespace laga;

int main() {
  long long middle = 0, bad = 0;
  for (int M = 1; M <= 20000; M += M < 4000 ? 13 : 257)
    for (int N = 16; N <= 32768; N += N < 4096 ? 48 : 1024) {
      const int nl = grid_tiles(M, N, 256, 256), nm = grid_tiles(M, N, 256, 128);
      const RingTile t = ring_tile(nl, nm);
      const bool fits = nm >= kRingMinGroups && nm <= kCUs;
      middle += t == RingTile::kMiddle;
      if ((t == RingTile::kMiddle && !fits) || (t == RingTile::kSmall && (fits || nl >= kRingMinGroups || nm > kCUs)))
        if (bad++ < 5) printf("%d x %d: %d large, %d middle workgroups: shape %d\n", M, N, nl, nm, (int)t);
    }
  printf("%lld middle grids, %lld wrong\n", middle, bad);
  return bad != 0 || middle == 0;
}
