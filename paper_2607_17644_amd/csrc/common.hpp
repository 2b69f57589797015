// Device helpers shared by the gfx950 kernels: element types, 8-element MFMA
// fragments, the 32x32 MFMA wrappers, LDS fragment reads and bf16 rounding.
//
// Fragment convention (all kernels): a 32x32 output block contracted over 16
// indices uses one "fragment" of 8 elements per lane for each operand. Lane l
// serves row/column (l % 32) of its operand and the contraction indices of
// half g = l / 32. For bf16 that is one v_mfma_f32_32x32x16_bf16; for fp32 it
// is eight v_mfma_f32_32x32x2_f32, the t-th taking element t of each fragment.
// The 16 accumulators of a lane hold the output column (l % 32) at rows
// (r / 4) * 8 + g * 4 + (r % 4), r = 0..15.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace laga {

typedef __bf16 bf16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(8 * sizeof(float)))) float f32x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short i16x4;

template <typename T> struct FragOf;
template <> struct FragOf<bf16> { using type = bf16x8; using half = bf16x4; };
template <> struct FragOf<float> { using type = f32x8; using half = f32x4; };
template <typename T> using frag_t = typename FragOf<T>::type;

__device__ __forceinline__ void mma(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma(f32x16& acc, const f32x8& a, const f32x8& b) {
#pragma unroll
  for (int t = 0; t < 8; ++t) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[t], b[t], acc, 0, 0, 0);
}

template <typename T> __device__ __forceinline__ T to_elem(float x);
template <> __device__ __forceinline__ bf16 to_elem<bf16>(float x) { return (bf16)x; }  // RNE
template <> __device__ __forceinline__ float to_elem<float>(float x) { return x; }
__device__ __forceinline__ float to_f32(bf16 x) { return (float)x; }
__device__ __forceinline__ float to_f32(float x) { return x; }

// 16-byte vector of elements used for global<->LDS staging (8 bf16 or 4 fp32).
typedef __attribute__((__vector_size__(16))) int chunk16;
template <typename T> struct Elems16 { static constexpr int n = 16 / sizeof(T); };

// Fragment of 8 contiguous elements from LDS (row-major, contraction along the row).
template <typename T>
__device__ __forceinline__ frag_t<T> lds_frag(const T* p) {
  return *reinterpret_cast<const frag_t<T>*>(p);
}

// Fragment whose 8 contraction indices run down a column of a row-major LDS
// tile X (pitch in elements): lane l returns X[ra + e][c] for e = 0..3 and
// X[rb + e][c] for e = 0..3, with c = c0 + (l % 32). ra and rb are per lane
// (they may depend on l / 32). For bf16 this uses ds_read_b64_tr_b16: each
// 16-lane group reads a 4 x 16 block, lane s of the group pointing at row
// (r + s / 4) and columns (4 * (s % 4)) .. +3 of the group's 16 columns.
template <typename T> struct TrRead;
template <> struct TrRead<bf16> {
  static __device__ __forceinline__ bf16x8 get(const bf16* X, int pitch, int ra, int rb, int c0) {
    const int l = threadIdx.x & 63;
    const int s = l & 15;
    const int col = c0 + 16 * ((l >> 4) & 1) + 4 * (s & 3);
    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
    const bf16* pa = X + (ra + (s >> 2)) * pitch + col;
    const bf16* pb = X + (rb + (s >> 2)) * pitch + col;
    bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(pa));
    bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(pb));
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};
template <> struct TrRead<float> {
  static __device__ __forceinline__ f32x8 get(const float* X, int pitch, int ra, int rb, int c0) {
    const int c = c0 + (threadIdx.x & 31);
    f32x8 f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      f[e] = X[(ra + e) * pitch + c];
      f[4 + e] = X[(rb + e) * pitch + c];
    }
    return f;
  }
};

// Accumulator rows r -> 8-element fragment used as the next MFMA's operand:
// rows 8*half .. 8*half+7 of the 16, i.e. for the 16 contraction indices
// 16*kk .. 16*kk+15 covered by accumulator block (kk / 2), half = kk % 2, the
// lane supplies indices {g*4 + e, 8 + g*4 + e} (e = 0..3) of that group of 16.
// Operands read with TrRead(ra = 16*kk + 4*g, rb = ra + 8) match this order.
template <typename T>
__device__ __forceinline__ frag_t<T> acc_to_frag(const f32x16& acc, int half) {
  frag_t<T> f;
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = to_elem<T>(acc[8 * half + e]);
  return f;
}
// bf16: one vector conversion, so that pairs map onto packed RNE conversions
template <>
__device__ __forceinline__ frag_t<bf16> acc_to_frag<bf16>(const f32x16& acc, int half) {
  typedef float f32x8 __attribute__((ext_vector_type(8)));
  f32x8 v;
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = acc[8 * half + e];
  return __builtin_convertvector(v, bf16x8);
}

__device__ __forceinline__ float wave_xor32_max(float x) {
  return fmaxf(x, __shfl_xor(x, 32));
}
__device__ __forceinline__ float wave_xor32_sum(float x) {
  return x + __shfl_xor(x, 32);
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }

// Direct global -> LDS copy of 16 bytes per lane (gfx950 global_load_lds_dwordx4):
// lane l's 16 bytes from `g` land at LDS address lds + 16 * l, where `lds` must be
// the same for every lane of the wave. Tracked by vmcnt like any global load.
//
// Two ways to issue it, chosen per source file with LAGA_LDS_DMA_ASM (defined before
// this header is included):
//   0: the compiler builtin. The compiler then models the copy as an access that may
//      also count on the LGKM counter, after which it waits for every LDS read with
//      lgkmcnt(0) (a full LDS round trip before each use).
//   1: inline assembly the compiler does not see as a memory access of its own: LDS
//      reads get exact lgkmcnt(N) waits. The kernel must then order the copies itself
//      (an explicit vmcnt wait and a barrier before a stage is read or refilled),
//      which every ring in this library does.
#ifndef LAGA_LDS_DMA_ASM
#define LAGA_LDS_DMA_ASM 0
#endif
// static: the definition differs between source files (see LAGA_LDS_DMA_ASM)
static __device__ __forceinline__ void g2lds16(const void* g, void* lds) {
#if LAGA_LDS_DMA_ASM
  // the low 32 bits of a generic pointer into LDS are its LDS address (an address
  // space cast would add a null check)
  const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(g), "s"(base) : "memory", "m0");
#else
  __builtin_amdgcn_global_load_lds(g, lds, 16, 0, 0);
#endif
}

// The same copy from a wave-uniform base plus a per-lane 32-bit byte offset (the
// scalar-base addressing form: one VGPR per lane instead of a 64-bit address).
#if LAGA_LDS_DMA_ASM
static __device__ __forceinline__ void g2lds16_so(const void* base, uint32_t off, void* lds) {
  const uint32_t m = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)lds);
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(m)
               : "memory", "m0");
}
#endif

// Workgroup barrier ordering LDS only: waits for this wave's LDS accesses, not for
// its global stores (__syncthreads also waits until every global store of the wave
// has completed). Direct global->LDS copies still need their own vmcnt wait first.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Wait until all of this wave's outstanding vector-memory loads (including direct
// global -> LDS copies) have completed.
__device__ __forceinline__ void wait_vmem() { __builtin_amdgcn_s_waitcnt(0); }

// Wait until at most N of this wave's vector-memory loads are outstanding (loads
// complete in issue order, so everything issued before the last N has landed).
// s_waitcnt immediate on gfx9: vmcnt in bits [3:0] and [15:14], expcnt [6:4] and
// lgkmcnt [11:8] left at their maxima (no wait on them).
template <int N>
__device__ __forceinline__ void wait_vmem_le() {
  static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// Ring of NS LDS stages fed by direct loads, at least F load instructions per wave
// per tile: before consuming a tile, wait until only the `ahead` tiles issued after
// it (ahead <= NS - 2) can still be in flight; with fewer tiles ahead (the end of
// the sweep) wait for everything.
template <int NS, int F>
__device__ __forceinline__ void ring_wait(int ahead) {
  static_assert(NS >= 2 && NS <= 4, "ring depth");
  if (NS >= 4 && ahead >= 2) wait_vmem_le<F * 2>();
  else if (NS >= 3 && ahead >= 1) wait_vmem_le<F>();
  else wait_vmem();
}

// ---------------------------------------------------------------- LDS tile layouts
// Bank model (64 banks x 4 bytes, measured on gfx950 with lane-pair probes): a read
// costs an extra pass whenever two lanes of one pass touch one bank at different
// addresses.
//   ds_read_b128: four passes of 16 lanes, pass = (lane bit 5, parity of lane bits
//     2..4), i.e. lanes {0-3, 12-15, 20-23, 24-27} and {4-11, 16-19, 28-31} for the
//     lower half-wave and likewise for the upper one.
//   ds_read_b64_tr_b16: two passes of 32 lanes (the half-waves).
// Read patterns of the kernels, by MFMA shape:
//   32x32x16 operands: (a) 16-byte row fragments, logical chunk c (even) of 32
//     consecutive rows in one half-wave and c+1 in the other; (b) transposing reads
//     of 4 chunks c..c+3 (c % 4 == 0) of 4 rows per 16 lanes, rows ra + {0, 8}.
//   16x16x32 operands: (a) 16-byte row fragments, chunk c + l/16 (c % 4 == 0) of 16
//     consecutive rows; (b) transposing reads of 2 chunks c, c+1 (c even) of 4 rows
//     per 16 lanes, rows {4G, 16 + 4G}.
//
// A "swizzled tile" is R rows x CPR 16-byte chunks stored without padding; logical
// chunk c of row r lives at physical chunk c ^ swz<CPR>(r) of that row. Without
// padding, a wave instruction of direct global->LDS loads fills 64 consecutive chunks.
// The XOR values below make both 32x32 patterns conflict-free (checked exhaustively
// under the model above; rows of 384 bytes start half-way round the banks on odd
// rows, rows of 256 bytes all start at bank 0). They are used for tiles read both
// ways (a) and (b); tiles read only one way use padded tiles (below).
template <int CPR> __device__ __forceinline__ int swz(int r);
template <> __device__ __forceinline__ int swz<16>(int r) {
  return ((r & 2) << 2) | ((r & 1) << 2) | ((r & 4) >> 1) | ((r >> 3) & 1);
}
template <> __device__ __forceinline__ int swz<24>(int r) {
  return ((r & 2) << 1) | ((r & 4) >> 1) | ((r >> 3) & 1);
}
template <> __device__ __forceinline__ int swz<8>(int r) {
  return ((r & 2) << 1) | ((r & 4) >> 1) | ((r >> 3) & 1);
}
template <> __device__ __forceinline__ int swz<4>(int r) { return (r >> 2) & 3; }

// Element offset of (row, element col) in a swizzled tile of CPR chunks per row.
template <typename T, int CPR>
__device__ __forceinline__ int swz_off(int row, int col) {
  constexpr int E = 16 / sizeof(T);
  return row * CPR * E + (((col / E) ^ swz<CPR>(row)) * E) + (col % E);
}

// 8-element row fragment (contraction along the row) at logical chunk c of `row`.
template <typename T, int CPR>
__device__ __forceinline__ frag_t<T> swz_frag(const T* tile, int row, int c) {
  constexpr int E = 16 / sizeof(T);
  return *reinterpret_cast<const frag_t<T>*>(tile + row * CPR * E + ((c ^ swz<CPR>(row)) * E));
}

// Transposing fragment from a swizzled bf16 tile: lane l gets X[ra + e][c0 + l%32]
// (e = 0..3) and X[rb + e][c0 + l%32] (e = 0..3); see TrRead for the lane layout.
template <int CPR>
__device__ __forceinline__ bf16x8 swz_tr_frag(const bf16* tile, int ra, int rb, int c0) {
  const int l = threadIdx.x & 63, s = l & 15;
  const int col = c0 + 16 * ((l >> 4) & 1) + 4 * (s & 3);  // element column of this lane's 8 bytes
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  const int r0 = ra + (s >> 2), r1 = rb + (s >> 2);
  const bf16* pa = tile + swz_off<bf16, CPR>(r0, col);
  const bf16* pb = tile + swz_off<bf16, CPR>(r1, col);
  bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(pa));
  bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(pb));
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// ---------------------------------------------------------------- padded tiles
// A "padded tile" holds NROWS rows of CPR 16-byte chunks at a pitch of P chunks (P - CPR
// chunks of padding at the end of each row). Unlike an XOR swizzle, padding keeps every
// LDS read of a lane at its own base address plus a compile-time offset, which saves
// registers and per-read address arithmetic. Conflict-free pitches under the bank
// model (checked exhaustively over chunk offsets and row blocks):
//   16x16x32 operands (both patterns): P % 4 == 2 (CPR 16 -> 18, CPR 24 -> 26);
//   32x32 16-byte row fragments only: P odd (CPR 8 -> 9, 16 -> 17, 24 -> 25);
//   32x32 transposing reads only: P % 8 == 4 (CPR 16 -> 20, 24 -> 28), or P = 4 for
//     tiles of exactly 32 columns (one 4-chunk group per row);
// no pitch serves both 32x32 patterns; a tile read both ways keeps the XOR swizzle.
//
// Chunks to allocate for a padded tile: NROWS * P rounded up to whole wave
// instructions of direct loads (64 chunks).
__host__ __device__ constexpr int pad_chunks(int nrows, int p) { return (nrows * p + 63) / 64 * 64; }

// Direct global->LDS fill by NW waves: wave instruction j covers physical chunks
// [64 j, 64 j + 64); lane i serves physical chunk p = 64 j + i, i.e. row p / P,
// chunk p % P, fetched from chunk_ptr(row, c). Lanes on padding, or past the last
// row (the allocation, NCH chunks, is rounded up to whole instructions), reload chunk
// 0 of their row / of row 0; those chunks are never read.
template <typename T, int NROWS, int CPR, int P, int NW, int NCH = pad_chunks(NROWS, P), typename ChunkPtr>
__device__ __forceinline__ void pad_fill_chunks(T* tile, int wave, int l, ChunkPtr chunk_ptr) {
  constexpr int E = 16 / sizeof(T);
  constexpr int NI = NCH / 64;
  static_assert(NCH % 64 == 0 && NCH >= NROWS * P, "allocation must be whole instructions");
#pragma unroll
  for (int j = wave; j < NI; j += NW) {
    const int p = j * 64 + l;
    int row = p / P, c = p % P;
    if (NI * 64 > NROWS * P && row >= NROWS) row = 0;
    g2lds16(chunk_ptr(row, c < CPR ? c : 0), tile + j * 64 * E);
  }
}

// Transposing fragment (32x32x16 lane layout, see TrRead) from a padded bf16 tile of
// pitch P chunks: lane l gets X[ra + e][c0 + l%32] and X[rb + e][c0 + l%32], e = 0..3.
template <int P>
__device__ __forceinline__ bf16x8 pad_tr_frag(const bf16* tile, int ra, int rb, int c0) {
  const int l = threadIdx.x & 63, s = l & 15;
  const int col = c0 + 16 * ((l >> 4) & 1) + 4 * (s & 3);
  typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
  const bf16* pa = tile + (ra + (s >> 2)) * P * 8 + col;
  const bf16* pb = tile + (rb + (s >> 2)) * P * 8 + col;
  bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(pa));
  bf16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(pb));
  return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// Swizzled-tile fill with the per-lane address arithmetic hoisted. For CPR = 4, 8 or 16 a
// load instruction covers 64 / CPR whole rows, and the swizzle depends on the row bits
// that the instruction index sets only through its residue modulo 2 (CPR 8) or 4
// (CPR 16; CPR 4: not at all); with NW a multiple of that, a lane's chunk permutation is the same in
// every instruction of its wave. So init() computes one element offset per lane, and
// a fill adds a wave-uniform row offset per instruction. Rows sit at a fixed element
// stride in global memory; a tile that crosses the end of the data (rows_valid <
// NROWS) takes the general path, clamping rows to rows_valid - 1.
template <typename T, int NROWS, int CPR, int NW>
struct SwzRowFill {
  static_assert(CPR == 4 || CPR == 8 || CPR == 16, "whole rows per load instruction");
  static constexpr int E = 16 / sizeof(T), RPI = 64 / CPR, NI = NROWS * CPR / 64;
  static_assert(NI * 64 == NROWS * CPR && NW % (CPR == 16 ? 4 : 2) == 0, "uniform chunk permutation per wave");
  int lane_off;
  __device__ __forceinline__ void init(int wave, int l, int stride) {
    const int rl = l / CPR;
    lane_off = rl * stride + ((l % CPR) ^ swz<CPR>(RPI * wave + rl)) * E;
  }
  __device__ __forceinline__ void fill(T* tile, int wave, int l, const T* base, int stride, int rows_valid) const {
    auto one = [&](int j) {
      if (rows_valid >= NROWS) {
        g2lds16(base + j * RPI * stride + lane_off, tile + j * 64 * E);
      } else {
        const int row = j * RPI + l / CPR, c = (l % CPR) ^ swz<CPR>(row);
        g2lds16(base + min(row, rows_valid - 1) * stride + c * E, tile + j * 64 * E);
      }
    };
    if constexpr (NI % NW == 0) {
      // the same number of instructions for every wave (wave < NW): no loop branches
#pragma unroll
      for (int i = 0; i < NI / NW; ++i) one(wave + i * NW);
    } else {
#pragma unroll
      for (int j = wave; j < NI; j += NW) one(j);
    }
  }
};

// Zero value of a 16-byte staging chunk.
__device__ __forceinline__ chunk16 zero_chunk() { chunk16 z = {0, 0, 0, 0}; return z; }

// XCD-aware ordering of a 1-D grid: the hardware deals consecutive workgroup
// ids round-robin over the 8 XCDs; this returns a "logical" id such that each
// XCD receives a contiguous range of logical ids (so work that shares data —
// same head, same tiles — lands on the same XCD and its L2). Needs n % 8 == 0
// to be a permutation; otherwise returns id unchanged.
__device__ __forceinline__ int xcd_remap(int id, int n) {
  constexpr int kXcd = 8;
  if (n % kXcd) return id;
  return (id % kXcd) * (n / kXcd) + id / kXcd;
}

// Workgroup id -> (head bh of B * H, block blk of nblk). Heads are taken in groups, and in a
// group each XCD (id % 8, as the hardware deals ids) keeps whole heads, for its L2, and takes
// their blocks in ascending order over all of them. With the causal mask a head's blocks
// differ in work and the caller numbers them heaviest first, so the heavy blocks of a group
// start before its light ones, which fill the gaps at its end (longest job first), and the
// last group ends the launch so. The groups are even, of at most about kOrderMasked
// (kOrderFull without the mask) workgroups per XCD: with fewer heads in a group the heavy
// blocks of one head run alone at its end, with more the heads' operands leave the L2 between
// two blocks of one head. The fused forward reads a head's 256 KB of W_kv_b again for every
// key tile, so its groups stay at 8 heads per XCD, half an L2, and without the mask at what
// the XCD's CUs run at once.
// Measured (us; one head after the other / all heads of the XCD in one group / this). Causal:
// forward, 128 heads x 8192 tokens 2651 / 2663 / 2504, 2 x 128 x 4096 1427 / 1512 / 1370, 64
// x 4096 377 / 328 / 328, 2 x 16 x 5001 274 / 252 / 252; dK/dV, 128 x 8192 6243 / 6442 / 5990,
// 64/32/64-wide 4 x 16 x 2000 122 / 108 / 107; fused forward, 128 x 4096 2063 / 2145 / 1815, 128
// x 2410 831 / 876 / 743, 2 x 128 x 745 248 / 294 / 225, 64 x 4096 1090 / 886 / 886. No mask:
// forward, 128 x 4096 1291 / 1305 / 1216; dK/dV there 2944 / 3214 / 2963; 64/32/64-wide, 64 x
// 4096 706 / 655 / 647; fused forward, 2 x 128 x 1569 1179 / 1276 / 1175. Groups of half the
// size, causal: forward at 64/32/64, 64 x 8192 706 -> 730; of twice the size, no mask: forward
// 128 x 4096 1305. Whole groups and an uneven rest: dK/dV, 64 x 5000 1175 -> 1236.
constexpr int kOrderMasked = 256, kOrderFull = 128;
struct BlockOrder {
  int heads, group, ids;  // B * H; heads of a group (a multiple of 8 unless it is the only one); its workgroups
};
constexpr int kOrderFusedMasked = 128, kOrderFusedFull = 32, kOrderFusedHeads = 8;  // the fused forward; heads per XCD
inline BlockOrder block_order(int nblk, int heads, int causal, bool fused_fwd = false) {
  const int size = fused_fwd ? (causal ? kOrderFusedMasked : kOrderFusedFull) : causal ? kOrderMasked : kOrderFull;
  int most = (size + nblk - 1) / nblk;
  if (fused_fwd && most > kOrderFusedHeads) most = kOrderFusedHeads;
  const int per_xcd = (heads + 7) / 8;
  const int groups = (per_xcd + most - 1) / most, even = 8 * ((per_xcd + groups - 1) / groups);
  const int group = heads < even ? heads : even;
  return {heads, group, group * nblk};
}
__host__ __device__ __forceinline__ void ordered_block(const BlockOrder& o, unsigned id, int& bh, int& blk) {
  unsigned j = id, h0 = 0;
  if (id >= (unsigned)o.ids) {  // (the division is most of the cost: the first group goes without)
    const unsigned grp = id / o.ids;
    j = id - grp * o.ids;
    h0 = grp * o.group;
  }
  const unsigned left = o.heads - h0;
  const unsigned hc = left < (unsigned)o.group ? left : o.group;
  if (hc % 8 == 0) {
    const unsigned c = hc / 8, i = j / 8;
    bh = h0 + j % 8 * c + i % c;
    blk = i / c;
  } else {  // heads shared between XCDs
    bh = h0 + j % hc;
    blk = j / hc;
  }
}

}  // namespace laga
