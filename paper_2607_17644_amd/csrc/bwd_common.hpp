// Declarations shared by the backward kernels (attn_bwd.hip, attn_bwd_dq.hip).
#pragma once
#include "common.hpp"

namespace laga {
namespace bwd {

// LDS row pitch (elements) of a tile read both with 16-byte row fragments and
// with transposing reads: for 16-bit types the pitch in dwords is chosen
// = 12, 28, 36 or 52 (mod 64) so that neither access pattern has bank
// conflicts; fp32 rows are padded to stay 32-byte aligned.
template <typename T>
constexpr int lds_pitch(int cols) {
  if (sizeof(T) == 4) return cols + 8;
  for (int pad = 8; pad < 136; pad += 16) {
    const int dw = ((cols + pad) / 2) % 64;
    if (dw == 12 || dw == 28 || dw == 36 || dw == 52) return cols + pad;
  }
  return cols + 8;
}

constexpr int round32(int x) { return (x + 31) / 32 * 32; }

struct BwdParams {
  const void* q;
  const void* k_pe;
  const void* kv;
  const void* dout;
  const float* lse;
  const float* delta;  // [B*H][S_pad]
  const float* lse2;   // [B*H][S_pad], lse * log2(e)
  int S_pad;
  void* dq;
  void* dkv;       // [B,S,H,DN+DV] element dtype
  void* dkv_lo;    // [B,S,H,DN+DV] bf16 low halves (bf16 only; else unused)
  float* dkpe_h;   // [B,S,H,DR] fp32
  int S, H, n_blocks;
  BlockOrder order;  // of the n_blocks blocks of every head (order_grid)
  float scale, scale_log2;
  int causal;
  // dS^T store (bf16 path with 192/128-wide heads): written by the key-stationary
  // pass, read by the dQ pass; see ds_tile_offset. ds_T = ceil(S / 32).
  void* ds;
  int ds_T;
  // K/V rebuilt on chip (kv_mode FUSED, bf16 with 192/128-wide heads): kv is unused and
  // each key's K_nope / V rows come from c_kv [B,S,d_c] and w_t = W_kv_b^T [H*(DN+DV), d_c]
  const void* c_kv;
  const void* w_t;
  int d_c;
};

// Launch grid of P.n_blocks blocks per head, in the order that it leaves in P.
inline dim3 order_grid(BwdParams& P, int B) {
  P.order = block_order(P.n_blocks, B * P.H, P.causal);
  return dim3(P.order.heads * P.n_blocks);
}

// dS^T store layout: for every (b, h) and query tile t of 32 rows, the keys that tile
// sees (32 (t + 1) with the causal mask, 32 T without) as rows of 32 bf16 values, one
// per query of the tile (key-major, 64-byte rows). Keys past S hold zeros. Within a row,
// query 8j + 4g + e (j < 4, g < 2, e < 4) sits at position 16g + 4j + e: the 16 queries
// one lane of the dK/dV kernel holds in its accumulator (column layout of the 32x32
// MFMA) are contiguous, so it writes them as two 16-byte stores.
__host__ __device__ constexpr int ds_query_of_position(int pos) {
  return 8 * ((pos >> 2) & 3) + 4 * (pos >> 4) + (pos & 3);
}
__host__ __device__ inline size_t ds_head_elems(int T, int causal) {
  return causal ? (size_t)512 * T * (T + 1) : (size_t)1024 * T * T;
}
__host__ __device__ inline size_t ds_tile_offset(int T, int causal, int bh, int t) {
  return (size_t)bh * ds_head_elems(T, causal) + (causal ? (size_t)512 * t * (t + 1) : (size_t)1024 * T * t);
}
__host__ __device__ inline int ds_tile_keys(int T, int causal, int t) { return causal ? 32 * (t + 1) : 32 * T; }

// Sequence lengths below which dK/dV splits the queries over pairs of waves (dkdv32_kernel with
// QS = 2; causal, full). A function of the sequence length and the mask alone, so that a
// head's gradients do not depend on the heads or batch elements beside it; the lines are set
// for the rank's share of 16 heads, and more (batch x heads) pay for it. A workgroup's first
// keys see every query, so with few workgroups that chain is the kernel's time, and the split
// halves it; but its step takes 13 % longer (copies one step ahead instead of two) and twice
// the workgroups pay 10 us of first loads and last stores. So every head count crosses
// elsewhere, and the lines are a compromise, no crossing of any: with the mask 16 heads cross
// between 2600 and 3000 tokens, 32 between 1000 and 1500, 64 between 300 and 600; without it,
// where every workgroup is as long, where the 64-key ones stop fitting the 256 CUs at once (16
// heads 1024 tokens, 8 heads 2048).
// Measured (us, QS = 1 / 2), causal, 16, 32, 64, 128 heads: 300 tokens 23 / 17, 24 / 18, 25 /
// 24, 31 / 40; 600 34 / 25, 35 / 28, 39 / 48, 71 / 93; 1000 50 / 35, 51 / 47, 74 / 88, 152 /
// 182; 1500 68 / 49, 76 / 84, 138 / 162, 281 / 332; 2048 88 / 72, 117 / 133, 235 / 262, 468 /
// 533; 2300 100 / 90, 145 / 161, 286 / 323, 569 / 653. No mask, 16, 32, 64 heads: 320 tokens
// 23 / 18, 23 / 18, 24 / 32; 640 35 / 26, 36 / 44, 63 / 70; 8, 16, 32 heads: 1024 49 / 34, 51 /
// 37, 60 / 69; 1200 57 / 38, 58 / 67, 105 / 102.
constexpr int kDkdvSplitMaxCausal = 2304, kDkdvSplitMaxFull = 1280;

// dkdv32_kernel with QS = 2 and the dS^T store: whether a wave (first key k0, T = ceil(S / 32)
// tiles) is certain to have issued the two dS^T stores of step j - 2 after the copies that it
// awaits at the start of step j, so that its wait may leave two operations in flight. Not
// before step 3 (no store yet, or none on the diagonal), and never in a wave whose keys all lie
// past the stored ones: without the mask and with an odd T that is the second half of the last
// 64-key workgroup, which stores nothing at all and copies rows that the first half reads.
__host__ __device__ constexpr bool dkdv_split_wait_counts(int T, int k0, int j) { return j > 2 && k0 < 32 * T; }

}  // namespace bwd
}  // namespace laga
