// MFMA GEMMs of the up-projection and its backward (gfx950).
//
//   reconstruct : kv[B*S, H*(d_nope+d_v)] = c_kv[B*S, d_c] @ W_kv_b     (Alg. 1 step 4)
//   dc          : dc_kv[B*S, d_c] = dKV[B*S, H*(d_nope+d_v)] @ W_kv_b^T   (fp32 out)
//   dW          : dW[d_c, H*(d_nope+d_v)] = c_kv^T @ dKV  (split over tokens,
//                 fixed-order reduction: deterministic)
//
// Each operand is either "k-contiguous" (stored [rows][K]) or "k-strided" (stored
// [K][rows]); both are staged into LDS as stored and strided operands are read back with
// transposing LDS reads, so there is no transpose pass anywhere. The output tile is
// computed as C^T = B^T A^T block by block, which puts 4 consecutive output columns in
// each lane's accumulators for vectorised stores.
//
// bf16: gemm_ring_kernel, an LDS ring of direct copies at three tile sizes, for any number
// of tokens; the reconstruct (a 512-long contraction writing 256 bytes per output row and
// head) runs large problems on a persistent variant that spreads each tile's stores over
// the next tile's MFMAs (gemm_stream_kernel). fp32: the register-staged gemm_kernel.
//
// Per output element the contraction runs over K in ascending 16-wide steps (one MFMA each;
// hi before lo where an operand is a pair) with fp32 accumulation. Tile shape, the persistent
// kernel and the shared launch of dc and dW are chosen by sizes that include N, the number of
// heads' columns: a column of kv or dW is bit-identical whatever N is only because every one
// of them accumulates an output in this same order, and because dW's token split does not
// depend on N. (dc_kv's contraction runs over the heads and may be split into partials summed
// in a fixed order.)
// direct global->LDS copies issued as inline assembly (exact LDS-read waits; the
// ring orders the copies with explicit waits and barriers)
#define LAGA_LDS_DMA_ASM 1
#include <type_traits>

#include "common.hpp"
#include "gemm_plan.hpp"
#include "kernels.hpp"

namespace laga {

namespace {

constexpr int kThreads = 256;

// xcd_remap for any n: the first n % 8 XCDs receive one id more. Partial row tiles give tile
// counts that are no multiple of 8, and workgroups that share operands then have to meet in
// one L2 all the same (dc, 10002 tokens, 128 x 128 tiles: 239 us without, 112 us with it).
__device__ __forceinline__ int xcd_remap_any(int id, int n) {
  const int x = id % 8;
  return x * (n / 8) + min(x, n % 8) + id / 8;
}

// One operand's tile of the fp32 kernel, staged through registers.
template <bool KSTRIDED, int ROWS, int BK>
struct OperandTile {
  using T = float;
  static constexpr int E = Elems16<T>::n;                      // elements per 16-byte chunk
  // k-contiguous rows: +8 elements keeps 16-byte fragment reads conflict-free and
  // fp32 rows 32-byte aligned; k-strided rows: +32 bytes for the transposing reads.
  static constexpr int PITCH = KSTRIDED ? ROWS + 8 : BK + 8;
  static constexpr int LDS_ELEMS = KSTRIDED ? BK * PITCH : ROWS * PITCH;
  static constexpr int CHUNKS = ROWS * BK / E;
  static constexpr int PER_THREAD = CHUNKS / kThreads;
  static_assert(CHUNKS % kThreads == 0, "tile must split evenly over the workgroup");

  chunk16 reg[PER_THREAD];

  // Global -> registers. rows [r0, r_end) valid, k [k0, k_end) valid; zero fill outside.
  __device__ __forceinline__ void load(const T* __restrict__ g, int ld, int r0, int r_end, int k0, int k_end) {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int c = tid + i * kThreads;
      int r, k;
      if (!KSTRIDED) { r = c / (BK / E); k = (c % (BK / E)) * E; }
      else { k = c / (ROWS / E); r = (c % (ROWS / E)) * E; }
      const int gr = r0 + r, gk = k0 + k;
      const bool ok = (gr < r_end) && (gk < k_end);
      const T* src = KSTRIDED ? g + (size_t)gk * ld + gr : g + (size_t)gr * ld + gk;
      reg[i] = ok ? *reinterpret_cast<const chunk16*>(src) : zero_chunk();
    }
  }
  __device__ __forceinline__ void store(T* s) const {
    const int tid = threadIdx.x;
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
      const int c = tid + i * kThreads;
      int r, k;
      if (!KSTRIDED) { r = c / (BK / E); k = (c % (BK / E)) * E; }
      else { k = c / (ROWS / E); r = (c % (ROWS / E)) * E; }
      T* dst = KSTRIDED ? s + k * PITCH + r : s + r * PITCH + k;
      *reinterpret_cast<chunk16*>(dst) = reg[i];
    }
  }
  // Fragment for the 32-row block starting at rb, contraction step ks.
  static __device__ __forceinline__ frag_t<T> frag(const T* s, int rb, int ks) {
    const int l = threadIdx.x & 63, g = l >> 5;
    if (!KSTRIDED) return lds_frag<T>(s + (rb + (l & 31)) * PITCH + ks * 16 + 8 * g);
    const int ra = ks * 16 + 8 * g;
    return TrRead<T>::get(s, PITCH, ra, ra + 4, rb);
  }
};

template <typename TO>
__device__ __forceinline__ void store4(TO* p, float a, float b, float c, float d);
template <>
__device__ __forceinline__ void store4<float>(float* p, float a, float b, float c, float d) {
  f32x4 v = {a, b, c, d};
  *reinterpret_cast<f32x4*>(p) = v;
}
template <>
__device__ __forceinline__ void store4<bf16>(bf16* p, float a, float b, float c, float d) {
  bf16x4 v = {(bf16)a, (bf16)b, (bf16)c, (bf16)d};
  *reinterpret_cast<bf16x4*>(p) = v;
}

// C (+ blockIdx.z * split_stride) [M][N] = A[M][K-range] B[K-range][N]
//
// A step is eight fp32 MFMAs per wave (0.25 us), shorter than a load from memory, so the
// global loads run kAhead steps ahead in registers (8 per step) and the steps alternate
// between two LDS buffers with one barrier each. Measured (us; one step ahead and one buffer /
// two / four steps ahead): 256 tokens, d_c 64, N 256: dc and dW 10.9 / 9.3 / 8.6 each; 2048
// tokens, d_c 512, N 4096: dc, dW and the reconstruct 272 / 264 / 249 together (four steps: 104
// TFLOP/s; the rest is the step's own chain, LDS store, barrier, LDS read, MFMA).
template <bool A_KS, bool B_KS, int BM, int BN, int BK>
__global__ __launch_bounds__(kThreads) void gemm_kernel(
    const float* __restrict__ A, const float* __restrict__ B, float* __restrict__ C,
    int M, int N, int K, int lda, int ldb, int ldc, int k_chunk, long long split_stride) {
  using T = float;
  using TA = OperandTile<A_KS, BM, BK>;
  using TB = OperandTile<B_KS, BN, BK>;
  constexpr int WM = BM / 64, WN = BN / 64;  // 32x32 blocks per wave along m and n
  constexpr int kAhead = 4;
  __shared__ __attribute__((aligned(16))) T sA[2][TA::LDS_ELEMS];
  __shared__ __attribute__((aligned(16))) T sB[2][TB::LDS_ELEMS];

  const int n_tiles = (N + BN - 1) / BN;
  const int m_tiles = (M + BM - 1) / BM;
  const int lin = xcd_remap(blockIdx.x, n_tiles * m_tiles);
  const int tn = lin % n_tiles, tm = lin / n_tiles;
  const int m0 = tm * BM, n0 = tn * BN;
  const int kb = blockIdx.z * k_chunk;
  const int ke = min(K, kb + k_chunk);

  const int wave = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 5;
  const int wm = wave & 1, wn = wave >> 1;

  f32x16 acc[WN][WM];
#pragma unroll
  for (int j = 0; j < WN; ++j)
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[j][i][r] = 0.f;

  TA ta[kAhead]; TB tb[kAhead];
  auto load = [&](int u, int k0) {  // zeros past ke
    ta[u].load(A, lda, m0, M, k0, ke);
    tb[u].load(B, ldb, n0, N, k0, ke);
  };
  auto store = [&](int u, int buf) {
    ta[u].store(sA[buf]); tb[u].store(sB[buf]);
  };
#pragma unroll
  for (int u = 0; u < kAhead; ++u) load(u, kb + u * BK);
  store(0, 0);
  load(0, kb + kAhead * BK);
  __syncthreads();
  const int n_steps = (ke - kb + BK - 1) / BK;
  for (int t0 = 0; t0 < n_steps; t0 += kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      if (t0 + u < n_steps) {  // step t0 + u: its buffer is u & 1, the next step's tile is in registers
        const int nu = (u + 1) % kAhead;
        store(nu, (u + 1) & 1);
        load(nu, kb + (t0 + u + 1 + kAhead) * BK);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
          frag_t<T> fa[WM], fb[WN];
#pragma unroll
          for (int i = 0; i < WM; ++i) fa[i] = TA::frag(sA[u & 1], (wm * WM + i) * 32, ks);
#pragma unroll
          for (int j = 0; j < WN; ++j) fb[j] = TB::frag(sB[u & 1], (wn * WN + j) * 32, ks);
#pragma unroll
          for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int i = 0; i < WM; ++i) mma(acc[j][i], fb[j], fa[i]);
        }
        __syncthreads();
      }
    }
  }

  float* Cz = C + blockIdx.z * split_stride;
#pragma unroll
  for (int j = 0; j < WN; ++j)
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      const int m = m0 + (wm * WM + i) * 32 + (l & 31);
      if (m >= M) continue;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int n = n0 + (wn * WN + j) * 32 + rr * 8 + g * 4;
        if (n < N)
          store4<float>(Cz + (size_t)m * ldc + n, acc[j][i][4 * rr], acc[j][i][4 * rr + 1],
                     acc[j][i][4 * rr + 2], acc[j][i][4 * rr + 3]);
      }
    }
}

// ------------------------------------------------------------------ ring tiles (bf16)
// A workgroup computes a BM x BN output tile on two waves per SIMD (eight waves, or four
// and two workgroups per CU), so that one wave's copies, LDS reads and barrier waits run
// beside the other's MFMAs: each wave owns 64 x 128, 128 x 64 (8 accumulator blocks of
// 32 x 32) or 64 x 64 (4 blocks) of it. The 256 x 256, 128 x 512 and 512 x 128 tiles read
// the least per product (the last two cover a whole 512-wide side, so the other, large
// operand is read from memory once); 256 x 128 and 128 x 128 are for problems with too few
// of those (launch_ring has the rule). The contraction advances 32 at a time through an LDS
// ring of NSLOT stages filled by direct global->LDS copies issued NSLOT - 1 stages ahead
// (a stage of MFMAs is shorter than the latency of a load from memory); one barrier per
// stage, between its two 16-wide steps, with the next stage's first operands read before
// the last MFMAs. Refills and waits are branch-free until the last NSLOT stages.
//
// Operand tiles are ROWS (the non-contraction index) x 32 contraction indices, stored
// unpadded as the copies fill them (a wave instruction fills 64 consecutive 16-byte
// chunks), with an XOR swizzle of the chunk index that keeps the operand reads
// conflict-free under the LDS bank model:
//   k-contiguous ([ROWS][32]: 4 chunks per row): chunk c of row r at c ^ ((r >> 2) & 3).
//     A row fragment read (32 rows, one chunk per half-wave) then covers 16 distinct
//     16-byte slots in each 16-lane pass.
//   k-strided ([32][ROWS]: ROWS / 8 chunks per k row, rows a multiple of 256 bytes):
//     chunk c of k row r at c ^ (4 (r & 3)). A transposing read covers 4 consecutive
//     k rows x 4 chunks per half-wave, which the XOR spreads over the four 64-byte
//     quarters of the banks.
// This lane's share of the copies of one operand tile (ROWS / 16 instructions, wave w
// of NWV issues w, w + NWV, ...).
template <bool KS, int ROWS, int NWV = 4>
struct GFill {
  static constexpr int NI = ROWS / 16, PER = NI / NWV, CPR = ROWS / 8;
  static_assert(PER * NWV == NI, "whole copy instructions per wave");
  uint32_t off[PER];  // byte offsets from the stage origin of the operand
  // r0: first row (column for KS) of the tile; rlim: number of rows (columns) in the operand.
  __device__ __forceinline__ void init(int wave, int l, int ld, int r0, int rlim) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int p = (wave + NWV * i) * 64 + l;
      if (!KS) {
        const int row = p >> 2, c = (p & 3) ^ ((row >> 2) & 3);
        off[i] = 2u * (uint32_t)(min(r0 + row, rlim - 1) * ld + c * 8);  // rows past the end read the last
      } else {
        const int kr = p / CPR, c = (p % CPR) ^ (4 * (kr & 3));
        off[i] = 2u * (uint32_t)(kr * ld + min(r0 + c * 8, rlim - 8));  // columns past the end likewise
      }
    }
  }
  __device__ __forceinline__ void fill(const bf16* stage_origin, bf16* tile, int wave) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) g2lds16_so(stage_origin, off[i], tile + (wave + NWV * i) * 512);
  }
  // a k-contiguous tile of which only the first `rows` rows exist (init with r0 = 0 and no
  // limit): the others copy row rows - 1
  __device__ __forceinline__ void fill_rows(const bf16* stage_origin, bf16* tile, int wave, int l, int ld,
                                            int rows) const {
    static_assert(!KS, "rows of a k-contiguous operand");
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int over = max((((wave + NWV * i) * 64 + l) >> 2) - (rows - 1), 0);
      g2lds16_so(stage_origin, off[i] - 2u * (uint32_t)(over * ld), tile + (wave + NWV * i) * 512);
    }
  }
  // a stage of which only the first `tail` contraction indices exist (a multiple of 8 for
  // k-contiguous tiles): the chunks of the others copy the stage's index 0 instead
  __device__ __forceinline__ void fill_part(const bf16* stage_origin, bf16* tile, int wave, int l, int ld,
                                            int tail) const {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int p = (wave + NWV * i) * 64 + l;
      uint32_t o = off[i];
      if (!KS) {
        const int c = (p & 3) ^ (((p >> 2) >> 2) & 3);
        if (c * 8 >= tail) o -= 2u * (uint32_t)(c * 8);
      } else {
        const int kr = p / CPR;
        if (kr >= tail) o -= 2u * (uint32_t)(kr * ld);
      }
      g2lds16_so(stage_origin, o, tile + (wave + NWV * i) * 512);
    }
  }
};

// Operand fragments of one wave's BW 32-row blocks (rows 32 BW wsel .. of the tile),
// contraction step ks (16 wide) of the stage.
template <bool KS, int ROWS, int BW = 4>
struct GRead {
  static_assert(BW == 2 || BW == 4, "two or four blocks per wave");
  int off[BW > 2 ? BW : 2];  // element offsets: k-contiguous uses [0..1] (per ks), k-strided one per block
  __device__ __forceinline__ void init(int l, int wsel) {
    const int g = l >> 5;
    if (!KS) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) off[ks] = (l & 31) * kGK + ((2 * ks + g) ^ ((l >> 2) & 3)) * 8;
    } else {
      // transposing read of k rows ra + s/4 (ra = 16 ks + 8 g; second half ra + 4) and
      // columns 32 b + 16 ((l >> 4) & 1) + 4 (s & 3) .. +3, s = l % 16, b = BW wsel + j;
      // logical chunk 4 b + lc of k row r sits at chunk 4 (b ^ (r & 3)) + lc, r & 3 = s / 4
      const int s = l & 15, j4 = s >> 2, lc = 2 * ((l >> 4) & 1) + ((s & 3) >> 1);
#pragma unroll
      for (int j = 0; j < BW; ++j)
        off[j] = j4 * ROWS + 8 * g * ROWS + (4 * ((BW * wsel + j) ^ j4) + lc) * 8 + 4 * (s & 1);
    }
  }
  __device__ __forceinline__ bf16x8 get(const bf16* tile, int wsel, int ks, int j) const {
    if (!KS) return *reinterpret_cast<const bf16x8*>(tile + (32 * BW * wsel + 32 * j) * kGK + off[ks]);
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const bf16* p = tile + off[j] + 16 * ks * ROWS;
    const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)p);
    const bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(p + 4 * ROWS));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

// C (+ blockIdx.z * split_stride) [M][N] = A[M][k range] B[k range][N], bf16 operands,
// fp32 accumulation, on NWV waves in a WGM x (NWV / WGM) grid of wave tiles. SPLIT: an
// operand is the sum of two bf16 tensors (1: A + X2, 2: B + X2; hi before lo per k-step). M and
// N are arbitrary for k-contiguous operands and at least 8 for k-strided ones (rows or columns
// past the end are copied from the last ones and not stored). The contraction of a split may
// end anywhere if both operands are k-strided, else at a multiple of 16: the last stage then
// copies in-bounds rows (k-strided) or chunks (k-contiguous) in the place of the missing
// ones, k-strided rows past the end are zeroed in LDS before they are read, and a second
// 16-wide step with nothing in it is left out.
constexpr int ring_stage(int BM, int BN, int SPLIT) {  // LDS elements of a stage
  return (BM + BN + (SPLIT == 1 ? BM : SPLIT == 2 ? BN : 0)) * kGK;
}
// A kernel here; in gemm_pair.hip the same body is a function that one kernel calls for dc and
// for dW (as a function called here too, its users' register allocation changes: dW 99 -> 109
// us at 2 x 5001 tokens).
template <int BM, int BN, int NWV, int WGM, int NSLOT, bool A_KS, bool B_KS, int SPLIT, typename TO>
#ifndef LAGA_GEMM_PAIR
__global__ __launch_bounds__(64 * NWV, NWV == 4 ? 2 : 1) void gemm_ring_kernel(
    const bf16* __restrict__ A, const bf16* __restrict__ B, const bf16* __restrict__ X2, TO* __restrict__ C,
    int M, int N, int K, int lda, int ldb, int ldc, int k_chunk, long long split_stride) {
  __shared__ __attribute__((aligned(16))) bf16 sm[NSLOT * ring_stage(BM, BN, SPLIT)];
  const int tile = blockIdx.x, split = blockIdx.z;
#else
__device__ __forceinline__ void gemm_ring_tile(bf16* sm, const int tile, const int split, const bf16* A,
                                               const bf16* B, const bf16* X2, TO* C, int M, int N, int K, int lda,
                                               int ldb, int ldc, int k_chunk, long long split_stride) {
#endif
  constexpr int WGN = NWV / WGM;                 // waves along n (WGM along m)
  constexpr int WTM = BM / WGM, WTN = BN / WGN;  // one wave's output tile
  constexpr int NI = WTM / 32, NJ = WTN / 32;    // its 32 x 32 blocks
  static_assert((NI == 2 || NI == 4) && (NJ == 2 || NJ == 4), "two or four blocks per wave and side");
  constexpr bool X_KS = SPLIT == 1 ? A_KS : B_KS;
  constexpr int XR = SPLIT == 1 ? BM : BN;
  constexpr int XB = SPLIT == 1 ? NI : NJ;       // X2 blocks per wave
  constexpr int TA = BM * kGK, TB = BN * kGK, TX = SPLIT ? XR * kGK : 0;
  constexpr int STAGE = TA + TB + TX;
  static_assert(STAGE == ring_stage(BM, BN, SPLIT), "stage size");

  const int n_tiles = (N + BN - 1) / BN, m_tiles = (M + BM - 1) / BM;
  const int lin = xcd_remap_any(tile, n_tiles * m_tiles);
  const int tn = lin % n_tiles, tm = lin / n_tiles;
  const int m0 = tm * BM, n0 = tn * BN;
  const int kb = split * k_chunk;
  const int klen = min(K, kb + k_chunk) - kb;
  const int nst = (klen + kGK - 1) / kGK;
  const int tail = klen - (nst - 1) * kGK;  // contraction indices of the last stage, 1 .. 32

  const int l = threadIdx.x & 63, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & (NWV - 1);
  const int wm = wave % WGM, wn = wave / WGM;

  GFill<A_KS, BM, NWV> fa;
  GFill<B_KS, BN, NWV> fb;
  GFill<X_KS, XR, NWV> fx;
  fa.init(wave, l, lda, m0, M);
  fb.init(wave, l, ldb, n0, N);
  if (SPLIT) fx.init(wave, l, SPLIT == 1 ? lda : ldb, SPLIT == 1 ? m0 : n0, SPLIT == 1 ? M : N);
  auto fill = [&](int t) {
    const int k = kb + t * kGK;
    bf16* st = sm + (t % NSLOT) * STAGE;
    fa.fill(A_KS ? A + (size_t)k * lda : A + k, st, wave);
    fb.fill(B_KS ? B + (size_t)k * ldb : B + k, st + TA, wave);
    if (SPLIT == 1) fx.fill(A_KS ? X2 + (size_t)k * lda : X2 + k, st + TA + TB, wave);
    if (SPLIT == 2) fx.fill(B_KS ? X2 + (size_t)k * ldb : X2 + k, st + TA + TB, wave);
  };
  auto fill_last = [&]() {  // stage nst - 1
    if (tail == kGK) return fill(nst - 1);
    const int k = kb + (nst - 1) * kGK;
    bf16* st = sm + ((nst - 1) % NSLOT) * STAGE;
    fa.fill_part(A_KS ? A + (size_t)k * lda : A + k, st, wave, l, lda, tail);
    fb.fill_part(B_KS ? B + (size_t)k * ldb : B + k, st + TA, wave, l, ldb, tail);
    if (SPLIT == 1) fx.fill_part(A_KS ? X2 + (size_t)k * lda : X2 + k, st + TA + TB, wave, l, lda, tail);
    if (SPLIT == 2) fx.fill_part(B_KS ? X2 + (size_t)k * ldb : X2 + k, st + TA + TB, wave, l, ldb, tail);
  };
  // after the copies of the last stage have landed in every wave: zeros for its k-strided
  // rows past the end of the contraction (both operands: no product of a missing index
  // meets a value of another one)
  auto zero_last = [&]() {
    if constexpr (A_KS && B_KS) {
      if (tail % 16 == 0) return;
      const int r1 = tail > 16 ? 32 : 16;
      bf16* st = sm + ((nst - 1) % NSLOT) * STAGE;
      auto zero = [&](bf16* tile, int rows) {
        for (int c = tail * (rows / 8) + (int)threadIdx.x; c < r1 * (rows / 8); c += 64 * NWV)
          *reinterpret_cast<chunk16*>(tile + c * 8) = zero_chunk();
      };
      zero(st, BM);
      zero(st + TA, BN);
      if (SPLIT) zero(st + TA + TB, XR);
      lds_barrier();
    }
  };
  constexpr int F = GFill<A_KS, BM, NWV>::PER + GFill<B_KS, BN, NWV>::PER + (SPLIT ? GFill<X_KS, XR, NWV>::PER : 0);
  auto wait_stage = [](int ahead) {
    if (ahead >= 3) wait_vmem_le<3 * F>();
    else if (ahead == 2) wait_vmem_le<2 * F>();
    else if (ahead == 1) wait_vmem_le<F>();
    else wait_vmem();
  };
  static_assert(NSLOT <= 4 && 3 * F < 64, "vmcnt range");

  GRead<A_KS, BM, NI> ra;
  GRead<B_KS, BN, NJ> rb;
  GRead<X_KS, XR, XB> rx;
  ra.init(l, wm);
  rb.init(l, wn);
  const int xsel = SPLIT == 1 ? wm : wn;
  if (SPLIT) rx.init(l, xsel);

  f32x16 acc[NJ][NI];  // [n block][m block]: C^T blocks, lane <-> m, 4 consecutive n per lane
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i) acc[j][i] = f32x16{};

  bf16x8 fA[2][NI], fB[2][NJ], fX[2][XB];
  auto read = [&](int t, int ks) {
    const bf16* st = sm + (t % NSLOT) * STAGE;
#pragma unroll
    for (int i = 0; i < NI; ++i) fA[ks][i] = ra.get(st, wm, ks, i);
#pragma unroll
    for (int j = 0; j < NJ; ++j) fB[ks][j] = rb.get(st + TA, wn, ks, j);
    if (SPLIT)
#pragma unroll
      for (int x = 0; x < XB; ++x) fX[ks][x] = rx.get(st + TA + TB, xsel, ks, x);
  };
  // every hi product of the step, then every lo one (per accumulator: hi before lo; an
  // MFMA that accumulates onto the one just issued would wait for its result)
  auto mmas = [&](int ks) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int i = 0; i < NI; ++i) mma(acc[j][i], fB[ks][j], fA[ks][i]);
    if (SPLIT)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int i = 0; i < NI; ++i) {
          if (SPLIT == 1) mma(acc[j][i], fB[ks][j], fX[ks][i]);
          if (SPLIT == 2) mma(acc[j][i], fX[ks][j], fA[ks][i]);
        }
  };

  const int npre = min(NSLOT, nst);
  for (int t = 0; t < npre; ++t) {
    if (t < nst - 1) fill(t);
    else fill_last();
  }
  wait_stage(npre - 1);
  lds_barrier();
  if (nst == 1) zero_last();
  read(0, 0);
  // refill: 0 a whole stage, 1 the last stage, 2 none left
  auto step = [&](int t, auto refill) {
    constexpr int R = decltype(refill)::value;
    read(t, 1);
    mmas(0);
    if constexpr (R < 2) wait_vmem_le<(NSLOT - 2) * F>();
    else wait_stage(nst - 2 - t);  // this wave's copies of stage t + 1 have landed
    lds_barrier();                 // ... everyone's; every read of stage t is done
    if constexpr (R == 0) fill(t + NSLOT);
    if constexpr (R == 1) fill_last();
    if constexpr (R == 2)
      if (t == nst - 2) zero_last();
    read(t + 1, 0);
    mmas(1);
  };
  int t = 0;
  for (; t + NSLOT < nst - 1; ++t) step(t, std::integral_constant<int, 0>{});
  if (t + NSLOT == nst - 1) step(t++, std::integral_constant<int, 1>{});
  for (; t < nst - 1; ++t) step(t, std::integral_constant<int, 2>{});
  if (tail > 16) read(nst - 1, 1);
  mmas(0);
  if (tail > 16) mmas(1);

  TO* Cz = C + split * split_stride;
#pragma unroll
  for (int j = 0; j < NJ; ++j)
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int m = m0 + WTM * wm + 32 * i + (l & 31);
      if (m >= M) continue;
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int n = n0 + WTN * wn + 32 * j + rr * 8 + g * 4;
        if (n < N)
          store4<TO>(Cz + (size_t)m * ldc + n, acc[j][i][4 * rr], acc[j][i][4 * rr + 1], acc[j][i][4 * rr + 2],
                     acc[j][i][4 * rr + 3]);
      }
    }
}

#ifndef LAGA_GEMM_PAIR

// ------------------------------------------------------------------ streamed large tiles (bf16 out)
// The 256 x 256 tile (no split, bf16 output) for a short contraction such as the
// latent's 512, where the 256 x 256 x 2-byte results of a tile take as long to write as
// its MFMAs take to compute, and a workgroup per tile writes them all at once while
// every other CU does the same. Here a persistent workgroup takes tiles q = blockIdx.x,
// + gridDim.x, ... and one LDS ring runs through all of them (the next tile's first
// stages are copied while the current one finishes). Eight waves, two per SIMD, each
// own 128 x 64 of the tile (8 accumulator blocks). A finished tile's accumulators are
// rounded to bf16 and paired across the two half-waves (v_permlane32_swap: 8
// consecutive columns per lane) into 16 16-byte stores per wave, issued one per stage
// over the 16 stages of the next tile, so the writes run at an even rate behind the
// MFMAs. Per output element the products are accumulated in the same order as in
// gemm_ring_kernel: the results are bitwise equal.
//
// Stores and copies share the in-order vmcnt counter: the stores issued in the last
// three stages are younger than the copies a stage waits for (those were issued three
// stages back) and older than none of them, so the ring's wait allows exactly that
// many more operations in flight.
constexpr int kStreamStoreStages = 16;  // stages over which a tile's stores are spread
constexpr int kStreamMaxK = 1024;       // longest contraction it is launched for


// RAGGED: the last row tile is partial (a variant of its own). It spills 69 registers (the
// whole-tile one 29, outside its stages): a store's 64-bit row address is reloaded from scratch
// in each of the sixteen store stages, and that wait drains the copies in flight. Measured (us,
// 16 heads, d_c 512): 16383 rows 82, 16384 75; 10002 rows 61, 9984 58.
template <int BM, int BN, bool A_KS, bool B_KS, bool RAGGED>
__global__ __launch_bounds__(512, 1) void gemm_stream_kernel(const bf16* __restrict__ A, const bf16* __restrict__ B,
                                                             bf16* __restrict__ C, int M, int N, int K, int lda,
                                                             int ldb, int ldc) {
  static_assert(BM == 256 && BN == 256 && !A_KS, "eight 128 x 64 waves; rows of A clamped at M");
  constexpr int WM = 2;  // waves along m (128 rows each); four along n (64 columns each)
  constexpr int NSLOT = 4;
  constexpr int TA = BM * kGK, TB = BN * kGK, STAGE = TA + TB;
  __shared__ __attribute__((aligned(16))) bf16 sm[NSLOT * STAGE];
  typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

  const int n_tiles = N / BN, n_items = n_tiles * (RAGGED ? (M + BM - 1) / BM : M / BM);
  const int G = gridDim.x, nst = K / kGK;                    // nst >= kStreamStoreStages
  const int mine = (n_items - 1 - (int)blockIdx.x) / G + 1;  // tiles of this workgroup
  const int total = mine * nst;                              // stages of this workgroup

  const int l = threadIdx.x & 63, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & 7;
  const int wm = wave % WM, wn = wave / WM;

  GFill<A_KS, BM, 8> fa;
  GFill<B_KS, BN, 8> fb;
  fa.init(wave, l, lda, 0, BM);  // offsets within a tile; the tile origin goes into the base
  fb.init(wave, l, ldb, 0, BN);
  auto tile_at = [&](int it, int& m0, int& n0) {
    const int id = (int)blockIdx.x + it * G;
    const int lin = RAGGED ? xcd_remap_any(id, n_items) : xcd_remap(id, n_items);
    n0 = (lin % n_tiles) * BN;
    m0 = (lin / n_tiles) * BM;
  };
  int f_loc = 0, f_it = 0, f_m0, f_n0;  // the next stage to copy
  tile_at(0, f_m0, f_n0);
  auto fill_next = [&](int slot) {
    const int k = f_loc * kGK;
    bf16* st = sm + slot * STAGE;
    if (!RAGGED || f_m0 + BM <= M) fa.fill(A + (size_t)f_m0 * lda + k, st, wave);
    else fa.fill_rows(A + (size_t)f_m0 * lda + k, st, wave, l, lda, M - f_m0);
    fb.fill(B_KS ? B + (size_t)k * ldb + f_n0 : B + (size_t)f_n0 * ldb + k, st + TA, wave);
    if (++f_loc == nst) {
      f_loc = 0;
      if (++f_it < mine) {
        tile_at(f_it, f_m0, f_n0);
      } else {  // past the last stage: copy it again into slots nobody reads any more
        f_it = mine - 1;
        f_loc = nst - 1;
      }
    }
  };
  constexpr int F = GFill<A_KS, BM, 8>::PER + GFill<B_KS, BN, 8>::PER;  // copies per wave and stage
  constexpr int Y = 3;  // stores younger than the copies a stage waits for, in steady state
  static_assert(3 * F + Y + 2 < 64, "vmcnt range");

  GRead<A_KS, BM, 4> ra;
  GRead<B_KS, BN, 2> rb;
  ra.init(l, wm);
  rb.init(l, wn);

  f32x16 acc[2][4];
  bf16x8 fA[2][4], fB[2][2];
  u32x4 pay[8][2];  // the previous tile's results, block (j, i) = 4 j + i, as stored
  auto read = [&](int slot, int ks) {
    const bf16* st = sm + slot * STAGE;
#pragma unroll
    for (int i = 0; i < 4; ++i) fA[ks][i] = ra.get(st, wm, ks, i);
#pragma unroll
    for (int j = 0; j < 2; ++j) fB[ks][j] = rb.get(st + TA, wn, ks, j);
  };
  auto mmas = [&](int ks, int j0, int j1) {
#pragma unroll
    for (int j = j0; j < j1; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) mma(acc[j][i], fB[ks][j], fA[ks][i]);
  };
  // Results of block (j, i) as two 16-byte stores per lane: lane half g takes columns
  // 16 p + 8 g .. + 7 (p = 0, 1) of its row; within a lane the 16 accumulators are 4
  // runs (rr) of 4 consecutive columns at 8 rr + 4 g, so runs 2p and 2p + 1 are
  // exchanged with the other half-wave.
  auto pack = [&](int j, int i, u32x4 (&out)[2]) {
    uint32_t x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
      const bf16x2 v = {(bf16)acc[j][i][2 * e], (bf16)acc[j][i][2 * e + 1]};
      x[e] = __builtin_bit_cast(uint32_t, v);
    }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      const auto r = __builtin_amdgcn_permlane32_swap(x[4 * p], x[4 * p + 2], false, false);
      const auto s = __builtin_amdgcn_permlane32_swap(x[4 * p + 1], x[4 * p + 3], false, false);
      out[p] = u32x4{r[0], s[0], r[1], s[1]};
    }
  };
  // half hh (columns 16 hh .. of the block) of block b: one 16-byte store per lane. Rows past
  // M were copied from row M - 1 and hold its results: they are stored there again (the same
  // bytes), so that every wave issues every store and the waits can count them.
  auto store = [&](const u32x4 (&v)[2], int m0, int n0, int b, int hh) {
    const int j = b >> 2, i = b & 3;
    const int m = m0 + 128 * wm + 32 * i + (l & 31);
    bf16* row = C + (size_t)(RAGGED ? min(m, M - 1) : m) * ldc + n0 + 64 * wn + 32 * j + 8 * g;
    *reinterpret_cast<u32x4*>(row + 16 * hh) = v[hh];
  };

  constexpr int RPS = (A_KS ? 8 : 4) + (B_KS ? 4 : 2);  // LDS reads per step
  constexpr int DS_READ = 0x100, MFMA = 0x008;
  // First half of stage t: step-1 reads interleaved with the step-0 MFMAs (which
  // restart every accumulator from zero in the first stage of a tile), then half of
  // the step-1 MFMAs.
  auto head = [&](int t, bool first) {
    read(t % NSLOT, 1);
    if (first) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[j][i] = f32x16{};
          mma(acc[j][i], fB[0][j], fA[0][i]);
        }
    } else {
      mmas(0, 0, 2);
    }
    mmas(1, 0, 1);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      __builtin_amdgcn_sched_group_barrier(DS_READ, RPS / 4, 0);
      __builtin_amdgcn_sched_group_barrier(MFMA, 2, 0);
    }
    __builtin_amdgcn_sched_group_barrier(MFMA, 4, 0);
    __builtin_amdgcn_sched_barrier(0);
  };
  // Second half of stage t: wait for stage t + 1, barrier, refill the slot of stage t,
  // read the step-0 operands of stage t + 1 with the other half of the step-1 MFMAs.
  // Every stage refills a slot (past the end with copies of the last stage), so two
  // stages of copies are always in flight behind the awaited one. With EXACT the wait
  // also leaves the Y stores of the last three stages in flight (they are younger than
  // the copies of stage t + 1, issued three stages back); otherwise it waits for them.
  // (s_waitcnt takes its count as an immediate: a count chosen at run time costs taken
  // branches every stage, which leave the matrix unit idle.)
  auto tail = [&](int t, auto exact) {
    if (decltype(exact)::value) wait_vmem_le<2 * F + Y>();
    else wait_vmem_le<2 * F>();
    lds_barrier();
    fill_next(t % NSLOT);
    __builtin_amdgcn_sched_barrier(0);
    read((t + 1) % NSLOT, 0);  // (after the last stage: a harmless read of a stale slot)
    mmas(1, 1, 2);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      __builtin_amdgcn_sched_group_barrier(DS_READ, RPS / 2, 0);
      __builtin_amdgcn_sched_group_barrier(MFMA, 2, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  for (int t = 0; t < NSLOT; ++t) fill_next(t);  // (total >= kStreamStoreStages > NSLOT)
  wait_vmem_le<(NSLOT - 1) * F>();
  lds_barrier();
  read(0, 0);

  int c_m0 = 0, c_n0 = 0;  // the tile being accumulated
  int e_m0 = 0, e_n0 = 0;  // the tile whose results are being stored
  int t = 0;
  // the first kStreamStoreStages stages of tile it, storing the previous tile's results
  auto first_stages = [&](int it, auto exact) {
#pragma unroll
    for (int s = 0; s < kStreamStoreStages; ++s, ++t) {
      head(t, s == 0);
      if (it > 0) store(pay[s >> 1], e_m0, e_n0, s >> 1, s & 1);
      tail(t, exact);
    }
  };
  for (int it = 0; it < mine; ++it) {
    tile_at(it, c_m0, c_n0);
    // From the third tile on (and with exactly kStreamStoreStages stages per tile) every
    // stage has stores of its own and of the two stages before it in flight.
    if (it >= 2 && nst == kStreamStoreStages) first_stages(it, std::true_type{});
    else first_stages(it, std::false_type{});
    for (int s = kStreamStoreStages; s < nst; ++s, ++t) {
      head(t, false);
      tail(t, std::false_type{});
    }
#pragma unroll
    for (int b = 0; b < 8; ++b) pack(b >> 2, b & 3, pay[b]);
    e_m0 = c_m0;
    e_n0 = c_n0;
  }
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    store(pay[b], e_m0, e_n0, b, 0);
    store(pay[b], e_m0, e_n0, b, 1);
  }
  wait_vmem();  // the surplus copies land before the workgroup's LDS is released
}

// The streamed kernel applies to whole column tiles (the last row tile may be partial)
// and at least kStreamStoreStages stages per tile.
bool gemm_stream_ok(int N, int K) { return N % 256 == 0 && K % kGK == 0 && K / kGK >= kStreamStoreStages; }

// dst[i] = sum_{s < nsplit} src[s * stride + i], in ascending s (float4 granularity).
__global__ __launch_bounds__(256) void split_reduce_kernel(const float* __restrict__ src, float* __restrict__ dst,
                                                           long long n4, int nsplit, long long stride) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n4) return;
  f32x4 s = reinterpret_cast<const f32x4*>(src)[i];
  for (int k = 1; k < nsplit; ++k) {
    f32x4 v = reinterpret_cast<const f32x4*>(src + k * stride)[i];
    s += v;
  }
  reinterpret_cast<f32x4*>(dst)[i] = s;
}

// fp32 tile of gemm_kernel
struct GemmCfg { static constexpr int BM = 64, BN = 64, BK = kFp32GK; };

// The backward's last launch: dc and dW from their split partials (ascending splits) and
// dk_pe[t, :] = sum over heads (ascending) of the per-head parts, 4 values per thread. One
// launch for the three: each alone is mostly launch and drain (5 to 7 us at 1000 tokens).
struct FinishArgs {
  const float *dc_part, *dw_part, *dkpe_h;
  float *dc, *dw, *dk_pe;
  long long n_dc, n_dw;          // float4 of dc, of dW (0: nothing to sum)
  int dc_splits, dw_splits, H, dr4;  // dr4: float4 per dk_pe row
  long long n_pe;                // float4 of dk_pe
  unsigned b_dc, b_dw;           // workgroups of dc, of dW; the rest dk_pe
};
__global__ __launch_bounds__(256) void finish_reduce_kernel(FinishArgs a) {
  const unsigned blk = blockIdx.x;
  auto sum = [](const float* src, float* dst, long long i, int n, long long stride4) {
    const f32x4* p = reinterpret_cast<const f32x4*>(src) + i;
    f32x4 s = p[0];
    for (int k = 1; k < n; ++k) s += p[k * stride4];
    reinterpret_cast<f32x4*>(dst)[i] = s;
  };
  if (blk < a.b_dc) {
    const long long i = (long long)blk * 256 + threadIdx.x;
    if (i < a.n_dc) sum(a.dc_part, a.dc, i, a.dc_splits, a.n_dc);
  } else if (blk < a.b_dc + a.b_dw) {
    const long long i = (long long)(blk - a.b_dc) * 256 + threadIdx.x;
    if (i < a.n_dw) sum(a.dw_part, a.dw, i, a.dw_splits, a.n_dw);
  } else {
    const long long i = (long long)(blk - a.b_dc - a.b_dw) * 256 + threadIdx.x;
    if (i >= a.n_pe) return;
    const long long row = i / a.dr4;
    const f32x4* p = reinterpret_cast<const f32x4*>(a.dkpe_h) + row * a.H * a.dr4 + i % a.dr4;
    f32x4 s = p[0];
    for (int h = 1; h < a.H; ++h) s += p[h * a.dr4];
    reinterpret_cast<f32x4*>(a.dk_pe)[i] = s;
  }
}

// C = A B over nz contraction ranges of k_chunk (C + z * M * N for range z); LBM x LBN: the large tile
template <int LBM, int LBN, bool A_KS, bool B_KS, int SPLIT, typename TO>
void launch_ring(const bf16* A, const bf16* B, const bf16* X2, TO* C, int M, int N, int K, int lda, int ldb, int ldc,
                 int k_chunk, int nz, hipStream_t st) {
  constexpr int NS = SPLIT ? 3 : 4;  // ring depth (LDS: at most 144 KB, 72 KB for 128 x 128)
  const long long stride = (long long)M * N;
  const int nl = grid_tiles(M, N, LBM, LBN), nm = grid_tiles(M, N, 256, 128);
  const RingTile tile = ring_tile(nl * nz, nm * nz);
  if (tile == RingTile::kLarge)
    gemm_ring_kernel<LBM, LBN, 8, (LBM <= LBN ? 2 : 4), NS, A_KS, B_KS, SPLIT, TO><<<dim3(nl, 1, nz), 512, 0, st>>>(
        A, B, X2, C, M, N, K, lda, ldb, ldc, k_chunk, stride);
  else if (tile == RingTile::kMiddle)
    gemm_ring_kernel<256, 128, 8, 4, NS, A_KS, B_KS, SPLIT, TO><<<dim3(nm, 1, nz), 512, 0, st>>>(
        A, B, X2, C, M, N, K, lda, ldb, ldc, k_chunk, stride);
  else
    gemm_ring_kernel<128, 128, 4, 2, NS, A_KS, B_KS, SPLIT, TO><<<dim3(grid_tiles(M, N, 128, 128), 1, nz), 256, 0, st>>>(
        A, B, X2, C, M, N, K, lda, ldb, ldc, k_chunk, stride);
}

}  // namespace

template <typename T>
hipError_t launch_reconstruct(const T* c, const T* w, T* kv, int M, int N, int K, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    // The persistent kernel where a tile's stores weigh as much as its products (short
    // contractions) and its last round of 256 x 256 tiles leaves at most a quarter of the
    // CUs idle. Measured (us, persistent / the ring's best; N = 4096, K = 512): 2048 rows
    // (128 tiles) 23 / 17, 4096 rows (256) 27 / 28, 5001 rows (320) 45 / 38, 8192 rows (512)
    // 45 / 53, 16384 rows 76 / 102; 8192 rows over K = 1024 72 / 75, over K = 2048 124 / 123,
    // over K = 4096 227 / 222; N = 7168, K = 16384: 2048 rows 450 / 419.
    const int tiles = grid_tiles(M, N, 256, 256), rounds = (tiles + kCUs - 1) / kCUs;
    if (gemm_stream_ok(N, K) && K <= kStreamMaxK && 3 * rounds * kCUs <= 4 * tiles) {
      const dim3 grid(tiles < kCUs ? tiles : kCUs);
      if (M % 256 == 0)
        gemm_stream_kernel<256, 256, false, true, false><<<grid, 512, 0, st>>>(c, w, kv, M, N, K, /*lda=*/K, /*ldb=*/N,
                                                                              /*ldc=*/N);
      else
        gemm_stream_kernel<256, 256, false, true, true><<<grid, 512, 0, st>>>(c, w, kv, M, N, K, /*lda=*/K, /*ldb=*/N,
                                                                             /*ldc=*/N);
    } else {
      launch_ring<256, 256, false, true, 0, bf16>(c, w, nullptr, kv, M, N, K, /*lda=*/K, /*ldb=*/N, /*ldc=*/N,
                                                  /*k_chunk=*/K, 1, st);
    }
  } else {
    using G = GemmCfg;
    gemm_kernel<false, true, G::BM, G::BN, G::BK><<<grid_tiles(M, N, G::BM, G::BN), kThreads, 0, st>>>(
        c, w, kv, M, N, K, /*lda=*/K, /*ldb=*/N, /*ldc=*/N, /*k_chunk=*/K, 0);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_finish(const FinishParams& f, hipStream_t st) {
  // dc[tokens][d_c] = (dKV + dKV_lo)[tokens][ncol] @ W^T, W stored [d_c][ncol] (k-contiguous);
  // dW[d_c][ncol] = c^T @ (dKV + dKV_lo), c stored [tokens][d_c] and dKV [tokens][ncol] (both
  // k-strided). Split contractions write partials that the last launch sums in a fixed order.
  const T *dkv = (const T*)f.dkv, *w = (const T*)f.w, *c = (const T*)f.c_kv;
  const int M = f.tokens, N = f.d_c, K = f.ncol;
  const int split = dw_split_tokens(M), nw = (int)dw_split_count(M);
  float* dw_part = f.partial;
  const DcPlan plan = dc_plan(M, N, K);
  float* dc_part = f.partial + (plan.pair ? dw_partial_elems(M, N, K) : 0);
  const long long sdc = (long long)M * N, sdw = (long long)N * K;
  int nz = 1;  // splits of dc
  if constexpr (sizeof(T) == 2) {
    const T* lo = (const T*)f.dkv_lo;
    const DcRanges r = dc_ranges(plan.splits, K, kGK);
    const int k_chunk = r.chunk;
    nz = r.n;
    float *dc = nz == 1 ? f.dc : dc_part, *dw = nw == 1 ? f.dw : dw_part;
    const int tdc = grid_tiles(M, N, 128, 128), tdw = grid_tiles(N, K, 128, 128);
    if (plan.pair) {
      const GemmPairArgs a = {dkv, lo, w, c, dc, dw, M, N, K, k_chunk, split, tdc, tdw, tdc * nz};
      launch_gemm_pair(a, tdc * nz + tdw * nw, st);
    } else {
      if (!plan.wide)
        gemm_ring_kernel<128, 128, 4, 2, 3, false, false, 1, float><<<dim3(tdc, 1, nz), 256, 0, st>>>(
            dkv, w, lo, dc, M, N, K, K, K, N, k_chunk, sdc);
      else if (N > 256)
        gemm_ring_kernel<128, 512, 8, 2, 3, false, false, 1, float><<<dim3(grid_tiles(M, N, 128, 512), 1, nz), 512, 0,
                                                                       st>>>(dkv, w, lo, dc, M, N, K, K, K, N, k_chunk,
                                                                             sdc);
      else
        gemm_ring_kernel<256, 256, 8, 2, 3, false, false, 1, float><<<dim3(grid_tiles(M, N, 256, 256), 1, nz), 512, 0,
                                                                       st>>>(dkv, w, lo, dc, M, N, K, K, K, N, k_chunk,
                                                                             sdc);
      if (nz > 1) {  // dW's partials take their place
        split_reduce_kernel<<<(unsigned)((sdc / 4 + 255) / 256), 256, 0, st>>>(dc_part, f.dc, sdc / 4, nz, sdc);
        nz = 1;
      }
      if (N > 256)
        launch_ring<512, 128, true, true, 2, float>(c, dkv, lo, dw, N, K, M, N, K, K, split, nw, st);
      else
        launch_ring<256, 256, true, true, 2, float>(c, dkv, lo, dw, N, K, M, N, K, K, split, nw, st);
    }
  } else {
    using G = GemmCfg;
    // dc's contraction in the plan's splits here too: one 64 x 64 tile per CU leaves the CUs
    // waiting on its loads (2048 tokens, 16 heads: 141 us in one range, 94 in four)
    const DcRanges r = dc_ranges(plan.splits, K, G::BK);
    const int k_chunk = r.chunk;
    nz = r.n;
    gemm_kernel<false, false, G::BM, G::BN, G::BK><<<dim3(grid_tiles(M, N, G::BM, G::BN), 1, nz), kThreads, 0,
                                                               st>>>(dkv, w, nz == 1 ? f.dc : dc_part, M, N, K, K, K, N,
                                                                     k_chunk, sdc);
    if (!plan.pair && nz > 1) {
      split_reduce_kernel<<<(unsigned)((sdc / 4 + 255) / 256), 256, 0, st>>>(dc_part, f.dc, sdc / 4, nz, sdc);
      nz = 1;
    }
    gemm_kernel<true, true, G::BM, G::BN, G::BK><<<dim3(grid_tiles(N, K, G::BM, G::BN), 1, nw), kThreads, 0,
                                                             st>>>(c, dkv, nw == 1 ? f.dw : dw_part, N, K, M, N, K, K,
                                                                   split, sdw);
  }
  FinishArgs a{};
  a.dc_part = dc_part; a.dw_part = dw_part; a.dkpe_h = f.dkpe_h; a.dc = f.dc; a.dw = f.dw; a.dk_pe = f.dk_pe;
  a.n_dc = nz > 1 ? sdc / 4 : 0;
  a.n_dw = nw > 1 ? sdw / 4 : 0;
  a.dc_splits = nz; a.dw_splits = nw; a.H = f.H; a.dr4 = f.d_rope / 4;
  a.n_pe = (long long)M * a.dr4;
  a.b_dc = (unsigned)((a.n_dc + 255) / 256);
  a.b_dw = (unsigned)((a.n_dw + 255) / 256);
  finish_reduce_kernel<<<a.b_dc + a.b_dw + (unsigned)((a.n_pe + 255) / 256), 256, 0, st>>>(a);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_gemm_nt(const T* a, const T* w, T* c, int M, int N, int K, hipStream_t st) {
  // c[M][N] = a[M][K] @ w^T, w stored [N][K] (both k-contiguous); element-dtype output
  if constexpr (sizeof(T) == 2) {
    launch_ring<256, 256, false, false, 0, bf16>(a, w, nullptr, c, M, N, K, K, K, N, K, 1, st);
  } else {
    using G = GemmCfg;
    gemm_kernel<false, false, G::BM, G::BN, G::BK><<<grid_tiles(M, N, G::BM, G::BN), kThreads, 0, st>>>(
        a, w, c, M, N, K, K, K, N, K, 0);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_gemm_tn(const T* a, const T* b, float* c, float* partial, int M, int N, int K, int nsplit,
                          hipStream_t st) {
  // c[M][N] = a^T @ b with a stored [K][M] and b [K][N] (both k-strided), fp32 output; the
  // contraction split into nsplit ranges of whole 32-index stages, summed in ascending order
  const int split = ((K + nsplit - 1) / nsplit + 31) / 32 * 32;
  const int nz = (K + split - 1) / split;
  float* target = nz == 1 ? c : partial;
  if constexpr (sizeof(T) == 2) {
    launch_ring<256, 256, true, true, 0, float>(a, b, nullptr, target, M, N, K, M, N, N, split, nz, st);
  } else {
    using G = GemmCfg;
    gemm_kernel<true, true, G::BM, G::BN, G::BK><<<dim3(grid_tiles(M, N, G::BM, G::BN), 1, nz), kThreads, 0,
                                                             st>>>(a, b, target, M, N, K, M, N, N, split,
                                                                   (long long)M * N);
  }
  if (nz > 1) {
    const long long n4 = (long long)M * N / 4;
    split_reduce_kernel<<<(unsigned)((n4 + 255) / 256), 256, 0, st>>>(partial, c, n4, nz, (long long)M * N);
  }
  return hipGetLastError();
}

template hipError_t launch_gemm_nt<bf16>(const bf16*, const bf16*, bf16*, int, int, int, hipStream_t);
template hipError_t launch_gemm_nt<float>(const float*, const float*, float*, int, int, int, hipStream_t);
template hipError_t launch_gemm_tn<bf16>(const bf16*, const bf16*, float*, float*, int, int, int, int, hipStream_t);
template hipError_t launch_gemm_tn<float>(const float*, const float*, float*, float*, int, int, int, int,
                                          hipStream_t);
template hipError_t launch_reconstruct<bf16>(const bf16*, const bf16*, bf16*, int, int, int, hipStream_t);
template hipError_t launch_reconstruct<float>(const float*, const float*, float*, int, int, int, hipStream_t);
template hipError_t launch_finish<bf16>(const FinishParams&, hipStream_t);
template hipError_t launch_finish<float>(const FinishParams&, hipStream_t);

#else
}  // namespace
#endif  // LAGA_GEMM_PAIR
}  // namespace laga
