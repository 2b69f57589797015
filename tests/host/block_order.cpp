// The order of the attention kernels' workgroups: every block of every head once; in a group
// whose heads deal out evenly an XCD keeps whole heads; a group's workgroups per XCD stay near
// the sizes that the order was measured at, so that the heads that an XCD works on at a time do
// not grow with the number of heads; and inside a group no block starts after one of a higher
// number on its XCD (heaviest first).
#include <stdio.h>

#include <vector>

#include "common.hpp"

int main() {
  long long ids = 0, bad = 0;
  auto fail = [&](const char* what, int nblk, int heads, int causal) {
    if (bad++ < 5) printf("%s: %d blocks, %d heads, causal %d\n", what, nblk, heads, causal);
  };
  for (int mode = 0; mode < 4; ++mode)
    for (int nblk : {1, 2, 3, 4, 7, 8, 16, 31, 32, 33, 63, 64, 100, 128, 129, 255, 256, 257, 512})
      for (int heads : {1, 2, 3, 4, 5, 7, 8, 9, 12, 15, 16, 17, 20, 24, 32, 60, 64, 100, 124, 128, 256, 520, 4096}) {
        const int causal = mode & 1, fused = mode >> 1;
        const laga::BlockOrder o = laga::block_order(nblk, heads, causal, fused);
        const int target = fused ? (causal ? laga::kOrderFusedMasked : laga::kOrderFusedFull)
                                 : causal ? laga::kOrderMasked : laga::kOrderFull;
        if (o.heads != heads || (o.group != heads && o.group % 8) || o.group > heads || o.ids != o.group * nblk)
          fail("group", nblk, heads, causal);
        if (o.ids >= 8 * (target + nblk)) fail("a group too large", nblk, heads, causal);
        // even groups, as few as the size allows
        const int wide = (target + nblk - 1) / nblk, groups = (heads + o.group - 1) / o.group;
        const int most = fused && wide > laga::kOrderFusedHeads ? laga::kOrderFusedHeads : wide;
        if (groups > ((heads + 7) / 8 + most - 1) / most) fail("too many groups", nblk, heads, causal);
        if (groups > 1 && heads - (groups - 1) * o.group + 8 * groups <= o.group) fail("an uneven rest", nblk, heads, causal);
        std::vector<int> seen((size_t)nblk * heads, 0), xcd(heads, -1);
        int prev[8] = {};
        for (int id = 0; id < heads * nblk; ++id, ++ids) {
          const int grp = id / o.ids, h0 = grp * o.group, left = heads - h0, in_group = left < o.group ? left : o.group;
          if (id % o.ids == 0)
            for (int& x : prev) x = 0;
          int bh = -1, blk = -1;
          laga::ordered_block(o, id, bh, blk);
          if (bh < h0 || bh >= h0 + in_group || blk < 0 || blk >= nblk || seen[(size_t)bh * nblk + blk]++) {
            fail("not a permutation", nblk, heads, causal);
            break;
          }
          const int x = id % 8;  // as the hardware deals ids
          if (in_group % 8 == 0 && xcd[bh] >= 0 && xcd[bh] != x) fail("a head on two XCDs", nblk, heads, causal);
          xcd[bh] = x;
          if (blk < prev[x]) fail("a block out of order", nblk, heads, causal);
          prev[x] = blk;
        }
        for (int n : seen)
          if (n != 1) fail("a block left out", nblk, heads, causal);
      }
  printf("%lld workgroups, %lld wrong\n", ids, bad);
  return bad != 0;
}
