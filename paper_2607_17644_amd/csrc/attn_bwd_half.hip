// Key-stationary dK / dV of the attention backward for bf16 with 64/32/64-wide heads
// (gfx950); see attn_bwd.hip for the whole backward. Built with MFMA results in VGPRs
// (the softmax arithmetic works on the S and dP accumulators).
#include <type_traits>

// direct global->LDS copies issued as inline assembly (exact LDS-read waits; the ring
// orders the copies with explicit waits and barriers)
#define LAGA_LDS_DMA_ASM 1
#include "common.hpp"
#include "kernels.hpp"
#include "bwd_common.hpp"

namespace laga {

using namespace bwd;

namespace {

// A wave owns 32 keys of one head: its K and V rows (operands of S = Q K^T and dP = dO V^T)
// and its dK^T / dV^T accumulators stay in registers (half the width of dkdv32_kernel's, so
// two waves fit on a SIMD and one wave's softmax runs beside the other's MFMAs: no software
// pipeline is needed). Per 32-query tile: 10 products of S and dP on row fragments, P and
// dZ in the accumulators' lanes, 10 products dV^T += dO^T P, dK^T += Q^T dZ on transposing
// reads. Tiles stream through a four-slot LDS ring of direct copies issued three tiles
// ahead: [Q nope 32 x 64 | Q rope 32 x 32 | dO 32 x 64 | lse2 | delta], 12 copy
// instructions, three per wave, each with its own wave-uniform base, row stride and LDS
// offset (no branch in a fill); past the last tile a fill copies that tile again into a
// slot nobody reads, so the wait is one immediate. What bounds it: MFMAs (20 x 32 cycles
// per tile and wave) and the softmax (16 exponentials of 16 cycles, about 100 other VALU
// instructions) share a SIMD between two waves, and LDS reads (20 KB per tile and wave)
// take a quarter of their rate. Measured at 4 x 2000 tokens, 16 heads (1024 workgroups, two
// per CU): 435 us for the generic kernel before, 136 us in head order, 110 us with the heavy
// blocks of an XCD's heads first.
template <int DN, int DR, int DV>
__global__ __launch_bounds__(256, 2) void dkdv_half_kernel(BwdParams P) {
  using T = bf16;
  constexpr int DQK = DN + DR, DKVH = DN + DV, NW = 4, BK = 32 * NW, BQ = 32, NS = 4, F = 3;
  constexpr int NKS = DQK / 16, NNS = DN / 16, NVS = DV / 16, NDK = DQK / 32, NDN = DN / 32, NDV = DV / 32;
  static_assert(DN == 64 && DR == 32 && DV == 64, "4 + 2 + 4 copy instructions per tile");
  constexpr int ON = 0, OR = ON + BQ * DN * 2, OO = OR + BQ * DR * 2, OL = OO + BQ * DV * 2, OD = OL + 1024;
  constexpr int STAGE = OD + 1024;  // bytes
  static_assert(NW * F == 12 && STAGE == 12 * 1024, "one copy instruction per KB");
  __shared__ __attribute__((aligned(16))) char sm[NS * STAGE];

  const T* __restrict__ q = (const T*)P.q;
  const T* __restrict__ kpe = (const T*)P.k_pe;
  const T* __restrict__ kv = (const T*)P.kv;
  const T* __restrict__ dout = (const T*)P.dout;
  const int S = P.S, H = P.H;

  int bh, kb;  // the first key blocks see the most queries
  ordered_block(P.order, blockIdx.x, bh, kb);
  const int b = bh / H, h = bh % H;

  const int l = threadIdx.x & 63, n = l & 31, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & (NW - 1);
  const int k0 = kb * BK + wave * 32;
  const int my_k = k0 + n;
  const bool key_ok = my_k < S;
  const size_t krow = (size_t)(b * S + (key_ok ? my_k : 0));
  const int qt_begin = P.causal ? kb * BK : 0;
  const int ntiles = (S - qt_begin + BQ - 1) / BQ;

  // copy instruction j = 3 wave + k of a tile: 0-3 Q nope, 4-5 Q rope, 6-9 dO, 10 lse2, 11 delta
  const char* base[F];    // of query 0 of this (b, h)
  uint32_t stride[F];     // bytes per query
  uint32_t off[F];        // this lane's bytes within the tile
  uint32_t row[F];        // this lane's query row (0 for lse2 / delta: their rows are padded)
#pragma unroll
  for (int k = 0; k < F; ++k) {
    const int j = wave * F + k;
    const size_t hq = (size_t)(b * S) * H + h;
    if (j < 6) {
      const bool rope = j >= 4;
      const int p = (rope ? j - 4 : j) * 64 + l;
      const int r = rope ? p >> 2 : p >> 3;
      const int c = rope ? (p & 3) ^ swz<4>(r) : (p & 7) ^ swz<8>(r);
      stride[k] = 2u * H * DQK;
      row[k] = r;
      off[k] = r * stride[k] + 16u * c;
      base[k] = (const char*)(q + hq * DQK + (rope ? DN : 0));
    } else if (j < 10) {
      const int p = (j - 6) * 64 + l, r = p >> 3, c = (p & 7) ^ swz<8>(r);
      stride[k] = 2u * H * DV;
      row[k] = r;
      off[k] = r * stride[k] + 16u * c;
      base[k] = (const char*)(dout + hq * DV);
    } else {
      stride[k] = 4u;
      row[k] = 0;
      off[k] = 16u * (l & 7);
      base[k] = (const char*)((j == 10 ? P.lse2 : P.delta) + (size_t)bh * P.S_pad);
    }
  }
  auto fill = [&](int slot, int j) {
    const int qt = qt_begin + min(j, ntiles - 1) * BQ;
    char* st = sm + slot * STAGE + wave * (F * 1024);
    if (qt + BQ <= S) {
#pragma unroll
      for (int k = 0; k < F; ++k) g2lds16_so(base[k] + (size_t)qt * stride[k], off[k], st + k * 1024);
    } else {  // rows past S read row S - 1 (masked below)
#pragma unroll
      for (int k = 0; k < F; ++k) {
        const uint32_t over = (uint32_t)max((int)row[k] - (S - 1 - qt), 0);
        g2lds16_so(base[k] + (size_t)qt * stride[k], off[k] - over * stride[k], st + k * 1024);
      }
    }
  };

  frag_t<T> kf[NKS], vf[NVS];
  {
    const T* kvr = kv + (krow * H + h) * DKVH;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const T* src = ks < NNS ? kvr + ks * 16 + 8 * g : kpe + krow * DR + (ks - NNS) * 16 + 8 * g;
      kf[ks] = *reinterpret_cast<const frag_t<T>*>(src);
      if (!key_ok) kf[ks] = frag_t<T>{};
    }
#pragma unroll
    for (int ks = 0; ks < NVS; ++ks) {
      vf[ks] = *reinterpret_cast<const frag_t<T>*>(kvr + DN + ks * 16 + 8 * g);
      if (!key_ok) vf[ks] = frag_t<T>{};
    }
  }
  f32x16 dk[NDK], dv[NDV];
#pragma unroll
  for (int i = 0; i < NDK; ++i) dk[i] = f32x16{};
#pragma unroll
  for (int i = 0; i < NDV; ++i) dv[i] = f32x16{};

  wait_vmem();  // the fragment loads: from here on only copies are counted
  fill(0, 0);
  fill(1, 1);
  fill(2, 2);
  constexpr int PF = 3;
  auto step = [&](auto sc, int j) {
    constexpr int ST = decltype(sc)::value;
    const int qt = qt_begin + j * BQ;
    wait_vmem_le<2 * F>();  // this wave's copies of tile j have landed
    lds_barrier();          // ... everyone's; every read of tile j - 1 is done
    fill((ST + 3) % NS, j + 3);
    if (k0 >= S || (P.causal && qt + BQ - 1 < k0)) return;  // wave-uniform: nothing to add
    const char* st = sm + ST * STAGE;
    const T* tn = (const T*)(st + ON);
    const T* tr = (const T*)(st + OR);
    const T* to = (const T*)(st + OO);
    const float* tl = (const float*)(st + OL);
    const float* td = (const float*)(st + OD);
    // products of S (i even < 2 NVS, i >= 2 NVS) and dP (i odd < 2 NVS), fragments read PF ahead
    auto a_is_s = [](int i) { return i >= 2 * NVS || (i & 1) == 0; };
    auto a_ks = [](int i) { return i >= 2 * NVS ? i - NVS : i >> 1; };
    auto a_frag = [&](int i) {
      const int ks = a_ks(i);
      if (!a_is_s(i)) return swz_frag<T, DV / 8>(to, n, 2 * ks + g);
      return ks < NNS ? swz_frag<T, DN / 8>(tn, n, 2 * ks + g) : swz_frag<T, DR / 8>(tr, n, 2 * (ks - NNS) + g);
    };
    constexpr int NA = NKS + NVS;
    f32x16 sa, dp;
    f32x4 lq[4], dl[4];
    {
      frag_t<T> ab[PF + 1];
#pragma unroll
      for (int i = 0; i < PF; ++i) ab[i] = a_frag(i);
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        lq[rr] = *reinterpret_cast<const f32x4*>(tl + rr * 8 + g * 4);
        dl[rr] = *reinterpret_cast<const f32x4*>(td + rr * 8 + g * 4);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NA; ++i) {
        if (i + PF < NA) ab[(i + PF) % (PF + 1)] = a_frag(i + PF);
        if (a_is_s(i))
          sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ab[i % (PF + 1)], kf[a_ks(i)], i == 0 ? f32x16{} : sa, 0, 0, 0);
        else
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ab[i % (PF + 1)], vf[a_ks(i)], i == 1 ? f32x16{} : dp, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if ((P.causal && qt < k0 + 31) || qt + BQ > S) {
      asm volatile("");  // a kept branch: only tiles on the diagonal or at the end
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int qi = qt + (r >> 2) * 8 + g * 4 + (r & 3);
        sa[r] = qi >= S || (P.causal && my_k > qi) ? -INFINITY : sa[r];
      }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float p = fast_exp2(__builtin_fmaf(sa[r], P.scale_log2, -lq[r >> 2][r & 3]));
      sa[r] = p;
      dp[r] = p * (dp[r] - dl[r >> 2][r & 3]);
    }
    bf16x8 pf[2], zf[2];
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      pf[kk] = acc_to_frag<T>(sa, kk);
      zf[kk] = acc_to_frag<T>(dp, kk);
    }
    // product i: query half kk = i / (NDK + NDV); blocks of dK^T, then of dV^T
    constexpr int NB = NDK + NDV, NC = 2 * NB;
    auto c_frag = [&](int i) {
      const int m = i % NB, ra = (i / NB) * 16 + 4 * g;
      if (m < NDN) return swz_tr_frag<DN / 8>(tn, ra, ra + 8, m * 32);
      if (m < NDK) return swz_tr_frag<DR / 8>(tr, ra, ra + 8, (m - NDN) * 32);
      return swz_tr_frag<DV / 8>(to, ra, ra + 8, (m - NDK) * 32);
    };
    {
      bf16x8 cb[PF + 1];
#pragma unroll
      for (int i = 0; i < PF; ++i) cb[i] = c_frag(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < NC; ++i) {
        if (i + PF < NC) cb[(i + PF) % (PF + 1)] = c_frag(i + PF);
        const int m = i % NB, kk = i / NB;
        if (m < NDK) mma(dk[m], cb[i % (PF + 1)], zf[kk]);
        else mma(dv[m - NDK], cb[i % (PF + 1)], pf[kk]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  };
  for (int j = 0; j < ntiles; j += NS) {
    step(std::integral_constant<int, 0>{}, j);
    if (j + 1 < ntiles) step(std::integral_constant<int, 1>{}, j + 1);
    if (j + 2 < ntiles) step(std::integral_constant<int, 2>{}, j + 2);
    if (j + 3 < ntiles) step(std::integral_constant<int, 3>{}, j + 3);
  }
  wait_vmem();  // the surplus copies land before the workgroup's LDS is released

  if (!key_ok) return;
  const size_t row_o = krow * H + h;
  T* dkvr = (T*)P.dkv + row_o * DKVH;
  T* dkvl = (T*)P.dkv_lo + row_o * DKVH;
  float* dper = P.dkpe_h + row_o * DR;
  // dKV as hi + lo: lo = bf16(x - hi) carries the next 8 bits for the GEMMs
  auto put = [&](int col, const f32x4& v) {
    bf16x4 hi, lo;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      hi[e] = to_elem<T>(v[e]);
      lo[e] = to_elem<T>(v[e] - to_f32(hi[e]));
    }
    *reinterpret_cast<bf16x4*>(dkvr + col) = hi;
    *reinterpret_cast<bf16x4*>(dkvl + col) = lo;
  };
#pragma unroll
  for (int db = 0; db < NDK; ++db)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int d = db * 32 + rr * 8 + g * 4;
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = dk[db][4 * rr + e] * P.scale;
      if (d >= DN) *reinterpret_cast<f32x4*>(dper + (d - DN)) = v;
      else put(d, v);
    }
#pragma unroll
  for (int db = 0; db < NDV; ++db)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = dv[db][4 * rr + e];
      put(DN + db * 32 + rr * 8 + g * 4, v);
    }
}

}  // namespace

hipError_t launch_dkdv_half(BwdParams P, int B, hipStream_t st) {
  P.n_blocks = (P.S + 127) / 128;
  const dim3 grid = order_grid(P, B);
  dkdv_half_kernel<64, 32, 64><<<grid, 256, 0, st>>>(P);
  return hipGetLastError();
}

}  // namespace laga
