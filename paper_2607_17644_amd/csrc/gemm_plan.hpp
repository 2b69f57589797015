// How the GEMMs of the up-projection's backward and of the output projection split their
// contractions, and the workspace that their partial sums take. Host arithmetic on sizes
// alone: the launches and the reported workspace both come from here.
#pragma once
#include <stddef.h>

#include <algorithm>

namespace laga {

constexpr int kCUs = 256;  // compute units of the gfx950 part (one large-tile workgroup each)
constexpr int kGK = 32;    // contraction per stage of the bf16 ring kernels
constexpr int kFp32GK = 16;  // contraction per step of the fp32 kernel

inline int grid_tiles(int M, int N, int BM, int BN) { return ((M + BM - 1) / BM) * ((N + BN - 1) / BN); }

// bf16 tile shapes of gemm_ring_kernel: "large" (the caller's BM x BN, 65536 outputs), "middle"
// 256 x 128 (both eight waves, one workgroup per CU) and "small" 128 x 128 (four waves, two
// workgroups per CU). The larger a tile, the less operand traffic per product, but fewer
// than kRingMinGroups workgroups leave CUs idle: the largest shape that gives them is
// launched, else the small one. A middle grid that does not fit the CUs at once takes a second
// round for a few workgroups and loses to the large one, which needs no second.
// Measured (us, large / middle / small, workgroups):
//   dW, 16 heads, d_c 512:  1000 tokens 36 (64) / 23 (128) / 20 (256);  2048 tokens 38 (128) /
//     30 (256) / 36 (512);  5001 tokens 59 (160) / 63 (320) / 69 (640);  16384 tokens 128 (256) /
//     137 (512) / 192 (1024)
//   y = out W_o (F = 16384, D = 7168):  300 tokens 306 (56) / 188 (112) / 136 (168);  1000 tokens
//     309 (112) / 246 (224) / 328 (448);  2048 tokens 419 (224) / 563 (448) / 697 (896)
//   kv, 16 heads, d_c 512:  2112 and 2304 tokens 22 (144) / 27 (288)
constexpr int kRingMinGroups = 160;
enum class RingTile { kLarge, kMiddle, kSmall };
inline RingTile ring_tile(int large, int middle) {  // workgroups of each
  if (large >= kRingMinGroups || middle > kCUs) return RingTile::kLarge;
  return middle >= kRingMinGroups ? RingTile::kMiddle : RingTile::kSmall;
}

// Tokens per split of the dW reduction over tokens: a function of the token count only
// (never of the head count), so each dW column is bit-identical whatever head shard
// computes it. 2048 for long sequences, down to 512 for short ones (enough workgroups).
inline int dw_split_tokens(int tokens) {
  int s = 2048;
  while (s > 512 && (tokens + s - 1) / s < 4) s /= 2;
  return s;
}
inline size_t dw_split_count(int tokens) {
  const int s = dw_split_tokens(tokens);
  return (size_t)((tokens + s - 1) / s);
}
inline size_t dw_partial_elems(int tokens, int d_c, int K) {
  return dw_split_count(tokens) > 1 ? dw_split_count(tokens) * (size_t)d_c * K : 0;
}

// dc's tiles: 128 x 128 (two workgroups per CU) while they fill the CUs no more than about
// once, with the contraction split where they don't (at least 512 indices per split); beyond,
// 128 x 512 (256 x 256 for d_c <= 256: the whole d_c side, so dKV is read once) over as many
// splits as fit the CUs and the partials of dW (so that dc adds nothing to the workspace).
// Measured (us with the reduction, 16 heads, d_c 512; 128 x 128 / 128 x 512, its splits in
// brackets): 1000 tokens 20 (8) / 31 (16), 2048 27 (4) / 38 (8), 4096 43 (2) / 50 (8), 8192
// 68 (1) / 76 (4), 10002 112 (1) / 96 (2), 16384 159 (1) / 135 (2).
inline bool dc_wide(int tokens, int d_c) { return grid_tiles(tokens, d_c, 128, 128) > kCUs + kCUs / 8; }
// dc and dW share a launch up to this many 128 x 128 workgroups (two per CU).
constexpr int kPairMaxGroups = 2 * kCUs;

// Partials that dc may have beside dW's (floats; 128 x 128 tiles, where one last launch sums
// both). The sum of both stays within max(dW's, the splits of a 512-workgroup grid of 128 x 128
// tiles - for token counts that are a multiple of 8 of a 256-workgroup grid of 65536-output
// ones -, at least 256 indices each): that is the workspace the library reported before the
// two shared a launch, so every problem that fits the fixed array of laga_attn_bwd_noalloc,
// or a workspace that a caller sized by it, keeps fitting. Nothing else hangs on tokens % 8.
inline size_t dc_partial_room(int tokens, int d_c, int K) {
  const bool aligned = tokens % 8 == 0;
  const int tiles = !aligned    ? grid_tiles(tokens, d_c, 128, 128)
                    : d_c > 256 ? grid_tiles(tokens, d_c, 128, 512)
                                : grid_tiles(tokens, d_c, 256, 256);
  const int want = aligned ? kCUs : 2 * kCUs, most = K >= 512 ? K / 256 : 1;
  const int n = std::min((want + tiles - 1) / tiles, most);
  const size_t cap = n > 1 ? (size_t)n * tokens * d_c : 0, dw = dw_partial_elems(tokens, d_c, K);
  return cap > dw ? cap - dw : 0;
}

// Splits of dc's contraction, and whether dc and dW share a launch (gemm_pair.hip): when the
// 128 x 128 tiles of both fit the chip at once and the workspace has room for the partials of
// both (a quarter fewer splits of dc than wanted is a fair price); the last launch then sums
// both. Otherwise dc's partials lie in the place of dW's and are summed right away, while they
// are in cache (2048 tokens, 16 heads: left to the last launch 5 us slower). Measured, the
// whole stage (us, apart / shared): 16 heads 100 tokens 26 / 17, 300 31 / 20, 1000 47 / 37, 8
// heads 1000 36 / 23; half-width heads, 4 x 2000 68 / 59.
struct DcPlan {
  bool wide, pair;
  int splits;  // the workspace holds this many partials
};
inline DcPlan dc_plan(int tokens, int d_c, int K) {
  DcPlan p{};
  p.wide = dc_wide(tokens, d_c);
  const int tiles = !p.wide     ? grid_tiles(tokens, d_c, 128, 128)
                    : d_c > 256 ? grid_tiles(tokens, d_c, 128, 512)
                                : grid_tiles(tokens, d_c, 256, 256);
  const size_t each = (size_t)tokens * d_c;
  int n = std::min(kCUs / tiles, K >= 1024 ? K / 512 : 1);
  if (p.wide) n = std::min(n, (int)(dw_partial_elems(tokens, d_c, K) / each));
  p.splits = n < 1 ? 1 : n;
  if (!p.wide) {
    const int fit = std::min(p.splits, (int)(dc_partial_room(tokens, d_c, K) / each));
    const int ns = p.splits == 1 || 4 * fit < 3 * p.splits ? p.splits : fit;
    p.pair = (p.splits == 1 || 4 * fit >= 3 * p.splits) &&
             tiles * ns + grid_tiles(d_c, K, 128, 128) * (int)dw_split_count(tokens) <= kPairMaxGroups;
    if (p.pair) p.splits = ns;
  }
  return p;
}
// The ranges that dc's contraction of K indices is launched in: `chunk` indices each (whole
// steps of the kernel; the last range may be shorter), `n` of them. The quotient is rounded
// up first, so that n never exceeds the splits: rounded down, a quotient that is a whole
// number of steps already leaves a remainder for one range more than there are partials.
struct DcRanges {
  int chunk, n;
};
inline DcRanges dc_ranges(int splits, int K, int step) {
  const int each = (K + splits - 1) / splits, chunk = (each + step - 1) / step * step;
  return {chunk, (K + chunk - 1) / chunk};
}

// Splits of gemm_tn's contraction of K indices for an M x N output (dw_o), each at least 512
// indices; a function of the shape only, and never more than were ever reported as workspace
// for it. fp32: enough for two 128 x 128 workgroups per CU. bf16: that many, and no more than
// for one 256 x 256 workgroup per CU. The latter alone used to decide where K is a multiple of
// 32, and the sum of its partials costs more than the workgroups gain (us, the whole backward
// of W_o, splits in brackets): T 2048, F 2048, D 7168 173 (2) / 132 (1); T 1024, F 2048, D 4096 79
// (2) / 59 (1); T 2048, F 2048, D 2048 65 (4) / 57 (2). From 4096 indices on it costs nothing (T
// 16384, F 2048, D 4096 486 (2) / 496 (1)) and stays as reported before, by K % 32.
inline int gemm_tn_splits(int M, int N, int K, int esize) {
  const int small = grid_tiles(M, N, 128, 128), large = grid_tiles(M, N, 256, 256);
  const int ns = (2 * kCUs + small - 1) / small, nl = (kCUs + large - 1) / large;
  const int n = esize == 4 ? ns : K < 4096 ? std::min(ns, nl) : K % kGK == 0 ? nl : ns;
  return std::max(1, std::min(n, (K + 511) / 512));
}

// Workspace of the split partials of dc_kv (its contraction, over the shard's heads x 256, is
// split so that the launch has enough workgroups; dc_kv sums over heads, so no bit-identity
// across head shards is asked of it) and of dW.
inline size_t gemm_partial_elems(int tokens, int d_c, int K) {
  const DcPlan p = dc_plan(tokens, d_c, K);
  const size_t dw = dw_partial_elems(tokens, d_c, K), dc = p.splits > 1 ? (size_t)p.splits * tokens * d_c : 0;
  return p.pair ? dw + dc : std::max(dw, dc);
}

}  // namespace laga
