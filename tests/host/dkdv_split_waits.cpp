// Every wait of the query-split dK/dV kernel against the stores that it leaves in flight: a
// wave that awaits the copies of step j, issued at the start of step j - 1, may leave as many
// operations in flight as the dS^T stores that it issued after them, in step j - 1 (for the
// query tile of step j - 2), and no more. All sequence lengths below the rule's lines, both
// masks, every wave of every workgroup and every step.
#include <stdio.h>

#include "bwd_common.hpp"

using namespace laga::bwd;

int main() {
  constexpr int QS = 2, BQ = 32, KW = 2, BK = 32 * KW;
  long long counted = 0, bad = 0;
  for (int causal = 0; causal < 2; ++causal)
    for (int S = 1; S < (causal ? kDkdvSplitMaxCausal : kDkdvSplitMaxFull); ++S) {
      const int T = (S + 31) / 32;
      for (int kb = 0; kb < (S + BK - 1) / BK; ++kb) {
        const int qt_begin = causal ? kb * BK : 0, steps = (S - qt_begin + BQ * QS - 1) / (BQ * QS);
        for (int wave = 0; wave < 2 * KW; ++wave) {
          const int k0 = kb * BK + (wave % KW) * 32, qw = wave / KW;
          for (int j = 0; j < steps; ++j) {
            int issued = 0;
            if (j >= 2) {
              const int t = (qt_begin + ((j - 2) * QS + qw) * BQ) / BQ;
              if (t < T && k0 < ds_tile_keys(T, causal, t)) issued = 2;  // lane 0 stores, so the wave does
            }
            const int allowed = dkdv_split_wait_counts(T, k0, j) ? 2 : 0;
            counted += allowed > 0;
            if (allowed > issued && bad++ < 5)
              printf("S %d causal %d: workgroup %d wave %d step %d leaves %d in flight, issued %d\n", S, causal, kb,
                     wave, j, allowed, issued);
          }
        }
      }
    }
  printf("%lld waits counted, %lld wrong\n", counted, bad);
  return bad != 0 || counted == 0;
}
