// The ranges that dc_kv's contraction is launched in against the partials that the workspace
// holds, for every token count up to 2100 and others beyond, latent width, head width and
// element type (contraction step), over head counts up to the library's limit.
#include <stdio.h>

#include "gemm_plan.hpp"

using namespace laga;

int main() {
  long long split = 0, bad = 0;
  auto one = [&](int tokens, int d_c, int K) {
    const DcPlan p = dc_plan(tokens, d_c, K);
    const size_t dw = dw_partial_elems(tokens, d_c, K), dc0 = p.pair ? dw : 0, have = gemm_partial_elems(tokens, d_c, K);
    for (int step : {kGK, kFp32GK}) {
      const DcRanges r = dc_ranges(p.splits, K, step);
      split += r.n > 1;
      const size_t need = r.n > 1 ? dc0 + (size_t)r.n * tokens * d_c : 0;
      const bool ok = r.chunk % step == 0 && r.n >= 1 && (long long)(r.n - 1) * r.chunk < K &&
                      (long long)r.n * r.chunk >= K && need <= have && dw <= have;
      if (!ok && bad++ < 5)
        printf("tokens %d d_c %d K %d step %d: %d ranges of %d for %d splits, %zu floats of %zu\n", tokens, d_c, K,
               step, r.n, r.chunk, p.splits, need, have);
    }
  };
  for (int tokens = 1; tokens < 40000; tokens += tokens < 2100 ? 1 : 501)
    for (int d_c = 32; d_c <= 1024; d_c += d_c < 256 ? 32 : 96)
      for (int w : {64, 128, 256})
        for (long long h = 1; h < 4096; h += h < 200 ? 1 : 13) {
          if (16ll * d_c * h * w >= 1ll << 31 || (long long)tokens * h * w * 3 / 2 >= 1ll << 31) break;
          one(tokens, d_c, (int)(h * w));
        }
  printf("%lld split contractions, %lld wrong\n", split, bad);
  return bad != 0 || split == 0;
}
