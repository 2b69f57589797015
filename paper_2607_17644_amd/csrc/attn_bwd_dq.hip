// dQ pass of the attention backward (gfx950); see attn_bwd.hip for the whole backward.
// Built with MFMA results kept in VGPRs (the dZ arithmetic on the dP accumulators of
// the recomputing kernel then needs no AGPR<->VGPR copies).
#include <type_traits>

// direct global->LDS copies issued as inline assembly (exact LDS-read waits; the
// rings order the copies with explicit waits and barriers)
#define LAGA_LDS_DMA_ASM 1
#include "common.hpp"
#include "kernels.hpp"
#include "bwd_common.hpp"

namespace laga {

using namespace bwd;

namespace {

// ------------------------------------------------------------------ dQ
// A workgroup of four waves owns 64 queries of one head: waves 0, 1 take the even 32-key tiles,
// waves 2, 3 the odd ones for the same queries (32 per wave; Q, dO and the dQ^T accumulators in
// registers), and the two partial sums meet in LDS at the end. As in the generic dK/dV kernel
// the work on a tile is split in two, A: S^T = K Q^T, P and half of dP^T = V dO^T, C: the rest of
// dP^T and dQ^T += K^T dS^T, phase p runs A of tile p on one pair beside C of tile p - 1 on the other, and
// tiles stream through three LDS slots of direct global->LDS copies. The chain of key tiles of
// the last queries is the kernel's time when there are no more workgroups than CUs; the pairs
// halve it. Before (128 queries per workgroup, each wave on every tile, tiles staged through
// registers) / now, us, fp32: 2048 tokens, 16 heads of 192/128 561 / 320, 32 heads x 4000 2326
// / 2282; 256 tokens, 4 heads of 48/32 27 / 20; 4 x 2000 tokens, 16 heads of 96/64 607 / 639 (the
// same step's dK/dV gains 105).
template <typename T, int DN, int DR, int DV>
__global__ __launch_bounds__(256, DN == 128 ? 1 : 2) void dq_kernel(BwdParams P) {
  constexpr int DQK = DN + DR, DKVH = DN + DV, DQK32 = round32(DQK), NDQ = DQK32 / 32;
  constexpr int BR = 64, BC = 32, NS = 3, E = Elems16<T>::n;
  constexpr int PK = lds_pitch<T>(DQK32), PV = lds_pitch<T>(DV);
  constexpr int KCH = DQK / E, VCH = DV / E, NCH = DN / E;  // chunks per row
  static_assert(KCH <= 64 && VCH <= 64, "one copy instruction per row");
  constexpr int TK = BC * PK, TV = BC * PV;
  __shared__ __attribute__((aligned(16))) T sm[NS * (TK + TV)];  // K slots, then V slots
  T* const sVm = sm + NS * TK;

  const T* __restrict__ q = (const T*)P.q;
  const T* __restrict__ kpe = (const T*)P.k_pe;
  const T* __restrict__ kv = (const T*)P.kv;
  const T* __restrict__ dout = (const T*)P.dout;
  const int S = P.S, H = P.H;

  int bh, qblk;
  ordered_block(P.order, blockIdx.x, bh, qblk);
  qblk = P.n_blocks - 1 - qblk;
  const int b = bh / H, h = bh % H;

  const int tid = threadIdx.x, l = tid & 63, n = l & 31, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
  const int qs = wave & 1, tw = wave >> 1;
  const int q0 = qblk * BR + qs * 32;
  const int my_q = q0 + n;
  const int kend = P.causal ? min(S, (qblk + 1) * BR) : S;
  const int nt = (kend + BC - 1) / BC;

  // zero the padding columns [DQK, DQK32) of every slot once: transposing reads touch them
  if (DQK32 > DQK)
    for (int i = tid; i < NS * BC * (DQK32 - DQK); i += 256)
      sm[(i / (DQK32 - DQK)) * PK + DQK + i % (DQK32 - DQK)] = to_elem<T>(0.f);

  frag_t<T> qf[DQK / 16], of[DV / 16];
  float lse2 = 0.f, dlt = 0.f;
  {
    const bool ok = my_q < S;
    const size_t base = (size_t)(b * S + (ok ? my_q : 0)) * H + h;
#pragma unroll
    for (int ks = 0; ks < DQK / 16; ++ks) {
      if (ok) qf[ks] = *reinterpret_cast<const frag_t<T>*>(q + base * DQK + ks * 16 + 8 * g);
      else
#pragma unroll
        for (int e = 0; e < 8; ++e) qf[ks][e] = to_elem<T>(0.f);
    }
#pragma unroll
    for (int ks = 0; ks < DV / 16; ++ks) {
      if (ok) of[ks] = *reinterpret_cast<const frag_t<T>*>(dout + base * DV + ks * 16 + 8 * g);
      else
#pragma unroll
        for (int e = 0; e < 8; ++e) of[ks][e] = to_elem<T>(0.f);
    }
    if (ok) {
      lse2 = P.lse2[(size_t)(b * H + h) * P.S_pad + my_q];
      dlt = P.delta[(size_t)(b * H + h) * P.S_pad + my_q];
    }
  }

  f32x16 dqa[NDQ];
#pragma unroll
  for (int i = 0; i < NDQ; ++i) dqa[i] = f32x16{};

  // Slot <- key tile j: wave w copies rows 8 w .. of K = [K_nope || k_pe] and of V, one
  // instruction per row (lane l chunk l); rows past S copy row S - 1 (masked below)
  const T* kvh = kv + ((size_t)(b * S) * H + h) * DKVH;
  const T* klane = l < NCH ? kvh + l * E : kpe + (size_t)(b * S) * DR + (l - NCH) * E;
  const uint32_t kstep = l < NCH ? (uint32_t)(H * DKVH) : (uint32_t)DR;
  auto fill = [&](int st, int j) {
    const int kt = j * BC;
    if (l < KCH)
#pragma unroll
      for (int i = 0; i < BC / 4; ++i) {
        const int r = wave * (BC / 4) + i;
        g2lds16(klane + (size_t)min(kt + r, S - 1) * kstep, sm + st * TK + r * PK);
      }
    if (l < VCH)
#pragma unroll
      for (int i = 0; i < BC / 4; ++i) {
        const int r = wave * (BC / 4) + i;
        g2lds16_so(kvh + (size_t)min(kt + r, S - 1) * H * DKVH + DN, 16u * l, sVm + st * TV + r * PV);
      }
  };
  // P and the first part of dP of the tile between its two halves: rows = keys (r/4)*8 + g*4 +
  // r%4, column = my query. dP's products are dealt so that both halves have as many.
  f32x16 sa, dp;
  constexpr int NV1 = (DV / 16 + 2 * NDQ - DQK / 16) / 2;
  static_assert(NV1 >= 0 && NV1 <= DV / 16, "dP steps of the first half");
  auto half_a = [&](int st, int j) {
    const T *sK = sm + st * TK, *sV = sVm + st * TV;
    const int kt = j * BC;
    sa = f32x16{};
    dp = f32x16{};
#pragma unroll
    for (int ks = 0; ks < DQK / 16; ++ks) mma(sa, lds_frag<T>(sK + n * PK + ks * 16 + 8 * g), qf[ks]);
#pragma unroll
    for (int ks = 0; ks < NV1; ++ks) mma(dp, lds_frag<T>(sV + n * PV + ks * 16 + 8 * g), of[ks]);
    const bool need_mask = (P.causal && kt + BC - 1 > q0) || (kt + BC > S);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float p = fast_exp2(sa[r] * P.scale_log2 - lse2);
      if (need_mask) {
        const int key = kt + (r >> 2) * 8 + g * 4 + (r & 3);
        if (key >= S || (P.causal && key > my_q)) p = 0.f;
      }
      sa[r] = p;
    }
  };
  auto half_c = [&](int st) {
    const T *sK = sm + st * TK, *sV = sVm + st * TV;
#pragma unroll
    for (int ks = NV1; ks < DV / 16; ++ks) mma(dp, lds_frag<T>(sV + n * PV + ks * 16 + 8 * g), of[ks]);
#pragma unroll
    for (int r = 0; r < 16; ++r) dp[r] = sa[r] * (dp[r] - dlt);
#pragma unroll
    for (int kk = 0; kk < BC / 16; ++kk) {
      const frag_t<T> zf = acc_to_frag<T>(dp, kk);
      const int ra = kk * 16 + 4 * g;
#pragma unroll
      for (int db = 0; db < NDQ; ++db) mma(dqa[db], TrRead<T>::get(sK, PK, ra, ra + 8, db * 32), zf);
    }
  };
  // start of phase p: tile p is there, tile p + 1 on its way into the slot of tile p - 2
  auto phase = [&](int p) {
    wait_vmem();      // this wave's copies of tile p have landed
    __syncthreads();  // everyone's; tile p - 2 is no longer read
    if (p + 1 < nt) fill((p + 1) % NS, p + 1);
  };
  fill(0, 0);
  if (tw) phase(0);
  for (int p = tw; p < nt; p += 2) {
    const bool on = q0 < S && (!P.causal || p * BC <= q0 + 31);  // wave-uniform
    phase(p);
    if (on) half_a(p % NS, p);
    phase(p + 1);
    if (on) half_c(p % NS);
  }
  if ((nt & 1) == tw) phase(nt);  // every wave goes through phases 0 .. nt

  // even tiles + odd tiles: the first wave of a pair takes blocks [0, NDQ / 2) of the other's
  // sum and stores them, the second the rest of the first's
  __syncthreads();
  constexpr int N0 = (NDQ + 1) / 2;
  static_assert(2 * NDQ * 4096 <= (int)sizeof(T) * NS * (TK + TV), "partials fit the slots");
  auto block = [&](int i) { return (float*)sm + (qs * NDQ + i) * 1024 + l * 4; };
#pragma unroll
  for (int i = 0; i < NDQ; ++i)
    if ((i < N0) == (tw == 1))
#pragma unroll
      for (int r = 0; r < 4; ++r)
        *reinterpret_cast<f32x4*>(block(i) + r * 256) = f32x4{dqa[i][4 * r], dqa[i][4 * r + 1], dqa[i][4 * r + 2], dqa[i][4 * r + 3]};
  __syncthreads();
  if (my_q >= S) return;
  T* dqr = (T*)P.dq + ((size_t)(b * S + my_q) * H + h) * DQK;
#pragma unroll
  for (int db = 0; db < NDQ; ++db) {
    if ((db < N0) != (tw == 0)) continue;
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int d = db * 32 + rr * 8 + g * 4;
      const f32x4 x = *reinterpret_cast<const f32x4*>(block(db) + rr * 256);
      if (d < DQK) {
        typename FragOf<T>::half v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = to_elem<T>((dqa[db][4 * rr + e] + x[e]) * P.scale);
        *reinterpret_cast<typename FragOf<T>::half*>(dqr + d) = v;
      }
    }
  }
}


// dQ recomputed without any S x S buffer (bf16, 192/128-wide heads): the forward's
// structure with dP and dS added. A workgroup of 8 waves owns 256 queries of one head (a
// wave 32, lane <-> query); 64-key tiles of K = [K_nope || k_pe] and V stream through a
// two-stage LDS ring of direct global->LDS loads into XOR-swizzled tiles. Per 32-key
// block: S^T = K Q^T and dP^T = V dO^T (A = K / V rows from LDS, B = the wave's Q and dO
// in registers, fragments read three products ahead), P^T = exp2(S^T scale_log2 - lse2),
// dS^T = P^T (dP^T - delta) in the accumulators' lanes, then dQ^T += K^T dS^T with K^T
// from transposing LDS reads and dS^T straight from the accumulators. The arithmetic
// per element is the key-stationary pass's (S and dP on the same MFMA products, the
// same exp2 argument, dS rounded once to bf16) and dQ sums the keys in ascending
// 16-wide steps, as the pass over the stored dS^T does: dq is bitwise equal to it.
template <int DN, int DR, int DV, int NW>
__global__ __launch_bounds__(64 * NW, DN == 128 ? 1 : 2) void dq_rec_kernel(BwdParams P) {
  using T = bf16;
  constexpr int DQK = DN + DR, DKVH = DN + DV, BC = 64, BR = 32 * NW;
  constexpr int KCPR = DN / 8, PCPR = DR / 8, VCPR = DV / 8;
  constexpr int NKS = DQK / 16, NVS = DV / 16, NDB = DQK / 32, NDN = DN / 32;
  static_assert(KCPR == VCPR && (KCPR == 16 || KCPR == 8) && (PCPR == 8 || PCPR == 4), "swizzled row widths");
  // two ring stages as distinct LDS objects (compile-time stage offsets in the reads)
  __shared__ __attribute__((aligned(16))) T sK0[BC * DN], sK1[BC * DN];
  __shared__ __attribute__((aligned(16))) T sP0[BC * DR], sP1[BC * DR];
  __shared__ __attribute__((aligned(16))) T sV0[BC * DV], sV1[BC * DV];

  const T* __restrict__ q = (const T*)P.q;
  const T* __restrict__ kpe = (const T*)P.k_pe;
  const T* __restrict__ kv = (const T*)P.kv;
  const T* __restrict__ dout = (const T*)P.dout;
  const int S = P.S, H = P.H;

  int bh, qblk;
  ordered_block(P.order, blockIdx.x, bh, qblk);
  qblk = P.n_blocks - 1 - qblk;
  const int b = bh / H, h = bh % H;

  const int tid = threadIdx.x, l = tid & 63, n = l & 31, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int q0 = qblk * BR + wave * 32;
  const int my_q = q0 + n;
  const int kend = P.causal ? min(S, (qblk + 1) * BR) : S;

  frag_t<T> qf[NKS], of[NVS];
  float lse2 = 0.f, dlt = 0.f;
  {
    const bool ok = my_q < S;
    const size_t base = (size_t)(b * S + (ok ? my_q : 0)) * H + h;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      qf[ks] = *reinterpret_cast<const frag_t<T>*>(q + base * DQK + ks * 16 + 8 * g);
      if (!ok) qf[ks] = frag_t<T>{};
    }
#pragma unroll
    for (int ks = 0; ks < NVS; ++ks) {
      of[ks] = *reinterpret_cast<const frag_t<T>*>(dout + base * DV + ks * 16 + 8 * g);
      if (!ok) of[ks] = frag_t<T>{};
    }
    if (ok) {
      lse2 = P.lse2[(size_t)(b * H + h) * P.S_pad + my_q];
      dlt = P.delta[(size_t)(b * H + h) * P.S_pad + my_q];
    }
  }
  f32x16 dqa[NDB];
#pragma unroll
  for (int i = 0; i < NDB; ++i) dqa[i] = f32x16{};

  // key rows past S are clamped to S - 1 (valid memory) and masked below
  SwzRowFill<T, BC, KCPR, NW> kfill, vfill;
  SwzRowFill<T, BC, PCPR, NW> pfill;
  kfill.init(wave, l, H * DKVH);
  vfill.init(wave, l, H * DKVH);
  pfill.init(wave, l, DR);
  auto fill_rows = [&](T* dk, T* dp, T* dv, int kt, int rows) {
    const T* kvb = kv + ((size_t)(b * S + kt) * H + h) * DKVH;
    kfill.fill(dk, wave, l, kvb, H * DKVH, rows);
    vfill.fill(dv, wave, l, kvb + DN, H * DKVH, rows);
    pfill.fill(dp, wave, l, kpe + (size_t)(b * S + kt) * DR, DR, rows);
  };
  // one branch per tile: whole tiles take the copies with no per-instruction row test
  auto fill = [&](T* dk, T* dp, T* dv, int kt) {
    if (S - kt >= BC) fill_rows(dk, dp, dv, kt, BC);
    else fill_rows(dk, dp, dv, kt, S - kt);
  };

  constexpr int PF = 3;
  const int ntiles = (kend + BC - 1) / BC;
  fill(sK0, sP0, sV0, 0);
  auto step = [&](auto stage, int it) {
    constexpr int ST = decltype(stage)::value;
    const int kt = it * BC;
    wait_vmem();      // this wave's loads of tile `it` have landed
    __syncthreads();  // ... and everyone's; the other stage is free
    if (it + 1 < ntiles) {
      if constexpr (ST == 0) fill(sK1, sP1, sV1, kt + BC);
      else fill(sK0, sP0, sV0, kt + BC);
    }
    if (P.causal && kt > q0 + 31) return;  // wave-uniform: every key of the tile is masked
    const T* tk = ST == 0 ? sK0 : sK1;
    const T* tp = ST == 0 ? sP0 : sP1;
    const T* tv = ST == 0 ? sV0 : sV1;
    const bool need_mask = (P.causal && kt + BC - 1 > q0) || (kt + BC > S);
#pragma unroll
    for (int kb = 0; kb < BC / 32; ++kb) {
      // product i of S^T (even i < 2 NVS and i >= 2 NVS: contraction step a_ks(i) of K) and
      // of dP^T (odd i < 2 NVS: step i / 2 of V), alternating accumulators
      auto a_is_s = [](int i) { return i >= 2 * NVS || (i & 1) == 0; };
      auto a_ks = [](int i) { return i >= 2 * NVS ? i - NVS : i >> 1; };
      auto a_frag = [&](int i) {
        const int ks = a_ks(i), row = kb * 32 + n;
        if (!a_is_s(i)) return swz_frag<T, VCPR>(tv, row, 2 * ks + g);
        return ks < DN / 16 ? swz_frag<T, KCPR>(tk, row, 2 * ks + g)
                            : swz_frag<T, PCPR>(tp, row, 2 * (ks - DN / 16) + g);
      };
      constexpr int NA = NKS + NVS;  // 20 products at 192/128-wide heads
      f32x16 sa, dp;
      {
        frag_t<T> ab[PF + 1];
#pragma unroll
        for (int i = 0; i < PF; ++i) ab[i] = a_frag(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NA; ++i) {
          if (i + PF < NA) ab[(i + PF) % (PF + 1)] = a_frag(i + PF);
          if (a_is_s(i))
            sa = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ab[i % (PF + 1)], qf[a_ks(i)], i == 0 ? f32x16{} : sa,
                                                         0, 0, 0);
          else
            dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ab[i % (PF + 1)], of[a_ks(i)], i == 1 ? f32x16{} : dp,
                                                         0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (need_mask) {
        asm volatile("");  // a kept branch: only tiles on the diagonal or at the end
        // live keys: accumulator row (r/4)*8 + r%4 of key block kb < klim - kt - 32 kb - 4 g
        const int lim = (P.causal ? min(S, my_q + 1) : S) - kt - 32 * kb - 4 * g;
#pragma unroll
        for (int r = 0; r < 16; ++r) sa[r] = (r >> 2) * 8 + (r & 3) < lim ? sa[r] : -INFINITY;
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = fast_exp2(__builtin_fmaf(sa[r], P.scale_log2, -lse2));
        dp[r] = p * (dp[r] - dlt);
      }
      bf16x8 zf[2];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) zf[kk] = acc_to_frag<T>(dp, kk);
      // dQ^T += K^T dS^T: product i = 16-key chunk kk = i / NDB, dQ block db = i % NDB
      auto k_tr = [&](int i) {
        const int kk = i / NDB, db = i % NDB, ra = kb * 32 + kk * 16 + 4 * g;
        return db < NDN ? swz_tr_frag<KCPR>(tk, ra, ra + 8, db * 32)
                        : swz_tr_frag<PCPR>(tp, ra, ra + 8, (db - NDN) * 32);
      };
      constexpr int NQ = 2 * NDB;
      {
        frag_t<T> kb_[PF + 1];
#pragma unroll
        for (int i = 0; i < PF; ++i) kb_[i] = k_tr(i);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
          if (i + PF < NQ) kb_[(i + PF) % (PF + 1)] = k_tr(i + PF);
          mma(dqa[i % NDB], kb_[i % (PF + 1)], zf[i / NDB]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  for (int it = 0; it < ntiles; it += 2) {
    step(std::integral_constant<int, 0>{}, it);
    if (it + 1 < ntiles) step(std::integral_constant<int, 1>{}, it + 1);
  }

  if (my_q >= S) return;
  T* dqr = (T*)P.dq + ((size_t)(b * S + my_q) * H + h) * DQK;
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = to_elem<T>(dqa[db][4 * rr + e] * P.scale);
      *reinterpret_cast<bf16x4*>(dqr + db * 32 + rr * 8 + g * 4) = v;
    }
}

// dQ from the stored dS^T (bf16, 192/128-wide heads): the key-stationary pass leaves
// dS^T = P * (dP - delta) of every causal (query tile, key) pair in the workspace, so
// this pass is a streaming product dQ^T (192 x 32 per wave) += K^T dS^T over the
// tile's keys, with no recomputation of S or dP. A workgroup of NW waves owns NW
// consecutive 32-query tiles of one head; key blocks of 32 stream through a four-stage
// LDS ring of direct global->LDS loads: the K_nope and k_pe rows of the block (shared,
// padded pitches of 20 and 12 chunks) and each wave's own 32 x 32 dS^T block (64-byte
// rows). Both MFMA operands come from transposing reads:
//   A = K^T (lane: head dim, 8 keys), B = dS^T (lane: query, the same 8 keys),
// the K fragments three products ahead in a pinned order. Every copy has a wave-uniform
// base and a constant byte offset per lane: with addresses worked out per copy the vector
// ALU spent as long on them as the matrix unit on the products. Every wave issues the same
// number of loads per stage (key blocks past a wave's queries load a dummy block that is
// not read), so the ring waits can count loads exactly.
// Bound: with few workgroups the chain of key blocks of the last query tiles (0.46 us a
// block at 2048 tokens), with many the dS^T stream (4.3 GB at 16384 tokens, 16 heads: 4.9
// TB/s). Measured before / now (16 heads, us): 1000 tokens 29 / 17, 2048 51 / 30, 4096
// 97 / 71, 2 x 5001 218 / 204, 8192 265 / 241. Two query tiles per wave, which used to win
// at 16384 tokens (one K fragment for two products), no longer does and is gone.
template <int DN, int DR, int DV, int NW>
__global__ __launch_bounds__(64 * NW, 1) void dq_ds_kernel(BwdParams P) {
  using T = bf16;
  constexpr int DQK = DN + DR, DKVH = DN + DV, KB = 32, NS = 4, PF = 3;
  constexpr int NCPR = DN / 8, NP = NCPR + 4, PP = DR / 8 + 4;  // K_nope and k_pe tiles, pitch % 8 == 4
  static_assert(NP % 8 == 4 && PP % 8 == 4, "conflict-free transposing reads");
  constexpr int NIN = pad_chunks(KB, NP) / 64, NI = NIN + pad_chunks(KB, PP) / 64;  // copy instructions
  static_assert(NI % NW == 0, "whole rounds of the workgroup");
  constexpr int F = NI / NW + 2;         // loads per wave per stage
  constexpr int DSE = NW * KB * 32;      // dS^T elements per stage
  __shared__ __attribute__((aligned(16))) T sK0[NI * 512], sK1[NI * 512], sK2[NI * 512], sK3[NI * 512];
  __shared__ __attribute__((aligned(16))) T sD0[DSE], sD1[DSE], sD2[DSE], sD3[DSE];

  const T* __restrict__ kpe = (const T*)P.k_pe;
  const T* __restrict__ kv = (const T*)P.kv;
  const T* __restrict__ ds = (const T*)P.ds;
  const int S = P.S, H = P.H, TT = P.ds_T;

  int bh, qblk;
  ordered_block(P.order, blockIdx.x, bh, qblk);
  qblk = P.n_blocks - 1 - qblk;
  const int b = bh / H, h = bh % H;

  const int l = threadIdx.x & 63, n = l & 31, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) & (NW - 1);
  const int t = qblk * NW + wave;  // this wave's query tile
  const bool wave_ok = t < TT;
  const int nk = wave_ok ? ds_tile_keys(TT, P.causal, t) : 0;  // keys stored for the tile
  const T* dtile = ds + (wave_ok ? ds_tile_offset(TT, P.causal, bh, t) : 0);
  const int kend = P.causal ? min(S, (qblk + 1) * NW * 32) : S;
  const int ntiles = (kend + KB - 1) / KB;

  f32x16 dqa[DQK / 32];
#pragma unroll
  for (int j = 0; j < DQK / 32; ++j) dqa[j] = f32x16{};

  // K copies: instruction j = wave + k NW covers 64 chunks of the K_nope tile (j < NIN) or of
  // the k_pe tile, from a wave-uniform row base plus this lane's constant byte offset (lanes
  // on padding reload chunk 0 of their row, past the last row that of row 0)
  constexpr int NKC = NI / NW;
  const char* kbase[NKC];  // key 0 of this (b, h)
  uint32_t krowb[NKC], koff[NKC], krow = 0;
#pragma unroll
  for (int k = 0; k < NKC; ++k) {
    const int j = wave + k * NW;
    const bool pe = j >= NIN;
    const int p = (pe ? j - NIN : j) * 64 + l;
    int r = pe ? p / PP : p / NP, c = pe ? p % PP : p % NP;
    if (r >= KB) r = 0;
    if (c >= (pe ? DR / 8 : NCPR)) c = 0;
    kbase[k] = pe ? (const char*)(kpe + (size_t)b * S * DR) : (const char*)(kv + ((size_t)(b * S) * H + h) * DKVH);
    krowb[k] = 2u * (pe ? (uint32_t)DR : (uint32_t)(H * DKVH));
    koff[k] = r * krowb[k] + 16u * c;
    krow |= (uint32_t)r << (5 * k);
  }
  static_assert(KB == 32 && NKC * 5 <= 32, "packed rows");
  auto fill = [&](T* dk, T* dd, int kt) {
    if (kt + KB <= S) {
#pragma unroll
      for (int k = 0; k < NKC; ++k) g2lds16_so(kbase[k] + (size_t)kt * krowb[k], koff[k], dk + (wave + k * NW) * 512);
    } else {  // rows past S read row S - 1 (their dS^T is zero or never read)
      const int k0 = min(kt, S - 1);
#pragma unroll
      for (int k = 0; k < NKC; ++k) {
        const int r = (int)((krow >> (5 * k)) & 31u), over = max(k0 + r - (S - 1), 0);
        g2lds16_so(kbase[k] + (size_t)k0 * krowb[k], koff[k] - over * krowb[k], dk + (wave + k * NW) * 512);
      }
    }
    const T* src = kt < nk ? dtile + (size_t)kt * 32 : dtile;  // dummy block when not stored
    T* dst = dd + wave * KB * 32;
    g2lds16_so(src, 16u * l, dst);
    g2lds16_so(src + 512, 16u * l, dst + 512);
  };

  // Every step refills a stage, past the last block with in-bounds dummies (clamped K
  // rows, the tile's first dS block) that nobody reads, so NS - 2 stages of loads are
  // always in flight behind the awaited one and the waits need no branch.
  fill(sK0, sD0, 0);
  fill(sK1, sD1, KB);
  fill(sK2, sD2, 2 * KB);
  auto step = [&](auto stage, int it) {
    constexpr int ST = decltype(stage)::value;
    const int kt = it * KB;
    wait_vmem_le<(NS - 2) * F>();  // this wave's loads of block `it` have landed
    lds_barrier();  // ... and everyone's; the stage filled next (read last at it - 1) is free
    {
      constexpr int NX = (ST + NS - 1) % NS;
      T* nk_ = NX == 0 ? sK0 : NX == 1 ? sK1 : NX == 2 ? sK2 : sK3;
      T* nd_ = NX == 0 ? sD0 : NX == 1 ? sD1 : NX == 2 ? sD2 : sD3;
      fill(nk_, nd_, kt + (NS - 1) * KB);
    }
    if (kt >= nk) return;  // wave-uniform: key blocks past a tile's queries hold no dS for it
    const T* tk = ST == 0 ? sK0 : ST == 1 ? sK1 : ST == 2 ? sK2 : sK3;
    const T* td = (ST == 0 ? sD0 : ST == 1 ? sD1 : ST == 2 ? sD2 : sD3) + wave * KB * 32;
    // product i: 16-key chunk i / NDB, 32-column block i % NDB of dQ
    constexpr int NDB = DQK / 32, NPR = KB / 16 * NDB;
    auto k_frag = [&](int i) {
      const int ra = (i / NDB) * 16 + 4 * g, db = i % NDB;
      return db < DN / 32 ? pad_tr_frag<NP>(tk, ra, ra + 8, db * 32)
                          : pad_tr_frag<PP>(tk + NIN * 512, ra, ra + 8, (db - DN / 32) * 32);
    };
    bf16x8 zf[KB / 16], kf[PF + 1];
#pragma unroll
    for (int kk = 0; kk < KB / 16; ++kk) zf[kk] = pad_tr_frag<4>(td, kk * 16 + 4 * g, kk * 16 + 4 * g + 8, 0);
#pragma unroll
    for (int i = 0; i < PF; ++i) kf[i] = k_frag(i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NPR; ++i) {
      if (i + PF < NPR) kf[(i + PF) % (PF + 1)] = k_frag(i + PF);
      mma(dqa[i % NDB], kf[i % (PF + 1)], zf[i / NDB]);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int it = 0; it < ntiles; it += NS) {
    step(std::integral_constant<int, 0>{}, it);
    if (it + 1 < ntiles) step(std::integral_constant<int, 1>{}, it + 1);
    if (it + 2 < ntiles) step(std::integral_constant<int, 2>{}, it + 2);
    if (it + 3 < ntiles) step(std::integral_constant<int, 3>{}, it + 3);
  }

  wait_vmem();  // the surplus loads land before the workgroup's LDS is released
  // accumulator column n holds the query stored at position n of the dS^T rows
  const int my_q = t * 32 + ds_query_of_position(n);
  if (!wave_ok || my_q >= S) return;
  T* dqr = (T*)P.dq + ((size_t)(b * S + my_q) * H + h) * DQK;
#pragma unroll
  for (int db = 0; db < DQK / 32; ++db)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = to_elem<T>(dqa[db][4 * rr + e] * P.scale);
      *reinterpret_cast<bf16x4*>(dqr + db * 32 + rr * 8 + g * 4) = v;
    }
}

// dQ from the stored dS^T with K/V rebuilt on chip (kv_mode FUSED; bf16, 192/128-wide
// heads): as dq_ds_kernel, but no per-head K exists in HBM, so each step's K tile is built
// in LDS: the K_nope rows of its 64 keys from the latent (KV^T = W_h^T c^T over d_c in
// ascending 16-wide steps, the up-projection GEMM's operand roles and rounding, so the
// tile equals the materialised kv bit for bit, and dq equals dq_ds_kernel's), the k_pe
// rows loaded as they are. Wave w rebuilds the 32 x 32 block (key half w / 4, K_nope
// columns 32 (w % 4) ..): every wave does the same 32 MFMAs per step, beside its 24 of
// the dQ product. The rebuild repeats for every query block of 256 rows (the price of a
// query-stationary pass: d_c * d_nope / (256 * d_qk) of its product flops, 1.33x).
template <int DN, int DR, int DV>
__global__ __launch_bounds__(512, 1) void dq_ds_fused_kernel(BwdParams P) {
  using T = bf16;
  constexpr int DQK = DN + DR, DKVH = DN + DV, NW = 8, KB = 64;
  constexpr int KP = DQK / 8 + 4;  // K tile pitch in 16-byte chunks (% 8 == 4: transposing reads)
  static_assert(DN == 4 * 32 && DR == 64, "four 32-column K_nope blocks, 64-wide k_pe");
  __shared__ __attribute__((aligned(16))) T sK[KB * KP * 8];
  __shared__ __attribute__((aligned(16))) T sD[NW * 2 * 32 * 32];

  const T* __restrict__ kpe = (const T*)P.k_pe;
  const T* __restrict__ ds = (const T*)P.ds;
  const int S = P.S, H = P.H, TT = P.ds_T, dc = P.d_c;

  int bh, qblk;
  ordered_block(P.order, blockIdx.x, bh, qblk);
  qblk = P.n_blocks - 1 - qblk;
  const int b = bh / H, h = bh % H;

  const int tid = threadIdx.x, wave = tid >> 6, l = tid & 63, n = l & 31, g = l >> 5;
  const int t = qblk * NW + wave;  // this wave's query tile
  const bool wave_ok = t < TT;
  const int nk = wave_ok ? ds_tile_keys(TT, P.causal, t) : 0;
  const T* dtile = ds + (wave_ok ? ds_tile_offset(TT, P.causal, bh, t) : 0);
  const int kend = P.causal ? min(S, (qblk + 1) * NW * 32) : S;
  const int nsteps = (kend + KB - 1) / KB;

  // this wave's share of the rebuild: key half rk, K_nope column block rb; W^T rows in the
  // order pi (bits 2 and 3 swapped) so that lane (n, g) holds columns 16 hh + 8 g + e (the
  // fragment-ordered copy of W^T holds them so: fragment (block rb, step ks) at wt + ks * 512)
  const int rk = wave >> 2, rb = wave & 3;
  const T* wt = (const T*)P.w_t + ((size_t)h * (DKVH / 32) + rb) * (dc / 16) * 512 + l * 8;
  const T* cg = (const T*)P.c_kv + (size_t)b * S * dc + 8 * g;

  f32x16 dqa[DQK / 32];
#pragma unroll
  for (int i = 0; i < DQK / 32; ++i) dqa[i] = f32x16{};

  for (int st = 0; st < nsteps; ++st) {
    const int kt = st * KB;
    __syncthreads();  // the previous step's reads of sK / sD are done
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {  // this wave's dS^T blocks of the step (a dummy when not stored)
      const int kb = kt + 32 * sub;
      const T* src = kb < nk ? dtile + (size_t)kb * 32 : dtile;
      g2lds16(src + l * 8, sD + (wave * 2 + sub) * 1024);
      g2lds16(src + 512 + l * 8, sD + (wave * 2 + sub) * 1024 + 512);
    }
    {  // k_pe rows: wave w copies keys 8 w .. 8 w + 7 (rows past S clamped: their dS is zero)
      const int r = wave * 8 + (l >> 3);
      const int key = min(kt + r, S - 1);
      const chunk16 v = *reinterpret_cast<const chunk16*>(kpe + (size_t)(b * S + key) * DR + (l & 7) * 8);
      *reinterpret_cast<chunk16*>(sK + r * KP * 8 + DN + (l & 7) * 8) = v;
    }
    {  // K_nope block (rk, rb)
      const int key = min(kt + 32 * rk + n, S - 1);
      const T* cr = cg + (size_t)key * dc;
      f32x16 acc = f32x16{};
      for (int k0 = 0; k0 < dc / 16; k0 += 8) {  // d_c % 128 == 0: 16 loads in flight, then 8 MFMAs
        frag_t<T> wa[8], cb[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          wa[j] = *reinterpret_cast<const frag_t<T>*>(wt + (k0 + j) * 512);
          cb[j] = *reinterpret_cast<const frag_t<T>*>(cr + (k0 + j) * 16);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) mma(acc, wa[j], cb[j]);
      }
      T* dst = sK + (32 * rk + n) * KP * 8 + rb * 32 + 8 * g;
      *reinterpret_cast<bf16x8*>(dst) = acc_to_frag<T>(acc, 0);
      *reinterpret_cast<bf16x8*>(dst + 16) = acc_to_frag<T>(acc, 1);
    }
    wait_vmem();
    __syncthreads();
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      if (kt + 32 * sub < nk) {  // wave-uniform: key blocks past the tile's queries hold no dS
        const T* tk = sK + 32 * sub * KP * 8;
        const T* td = sD + (wave * 2 + sub) * 1024;
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int ra = kk * 16 + 4 * g;
          const bf16x8 zf = pad_tr_frag<4>(td, ra, ra + 8, 0);
#pragma unroll
          for (int db = 0; db < DQK / 32; ++db) mma(dqa[db], pad_tr_frag<KP>(tk, ra, ra + 8, db * 32), zf);
        }
      }
    }
  }

  const int my_q = t * 32 + ds_query_of_position(n);
  if (!wave_ok || my_q >= S) return;
  T* dqr = (T*)P.dq + ((size_t)(b * S + my_q) * H + h) * DQK;
#pragma unroll
  for (int db = 0; db < DQK / 32; ++db)
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      bf16x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = to_elem<T>(dqa[db][4 * rr + e] * P.scale);
      *reinterpret_cast<bf16x4*>(dqr + db * 32 + rr * 8 + g * 4) = v;
    }
}

// The same product with the K_nope rebuild organised around its operand traffic (d_c =
// 512): 4 waves (one per SIMD); wave w owns K_nope column block w and keeps its 32 rows of
// W_h^T (pi-ordered, 32 fragments) in registers for the whole kernel, and TPW
// consecutive 32-query tiles (the rebuilt K tile serves 32 * 4 * TPW queries, which sets
// the rebuild's share of the work: 1.33x the dQ products at TPW = 2). Per 64-key step the
// latent rows are copied once into LDS (direct loads, one 1 KB row per wave instruction,
// rows padded to 65 chunks: conflict-free row fragments) and each wave rebuilds its
// column block for both 32-key halves (two independent accumulator chains), so W_h^T is
// read once per workgroup and each latent row once per step. The copies of step s + 1
// (latent rows into the then free sC, dS^T blocks into the other of two sD stages, k_pe
// rows into registers) are issued right after the rebuild of step s, so that they land
// while the step's dQ products run. Operand roles, contraction order and rounding are
// those of dq_ds_fused_kernel: the K tile and dq are the same bit for bit.
template <int DN, int DR, int DV, int DC, int TPW>
__global__ __launch_bounds__(256, 1) void dq_ds_fused2_kernel(BwdParams P) {
  using T = bf16;
  constexpr int DQK = DN + DR, DKVH = DN + DV, NW = 4, KB = 64, NKS = DC / 16;
  constexpr int KP = DQK / 8 + 4;  // K tile pitch in 16-byte chunks (% 8 == 4: transposing reads)
  constexpr int CP = DC / 8 + 1;   // latent row pitch in chunks (odd: row fragments conflict-free)
  constexpr int DSW = TPW * 2 * 32 * 32;  // dS^T elements per wave and step
  static_assert(DN == NW * 32 && DR == 64 && DC == 64 * 8, "one 32-column K_nope block per wave; a latent row per copy");
  static_assert(TPW == 1 || TPW == 2, "one or two query tiles per wave");
  static_assert(KB * DR / 8 == 64 * NW * 2, "two k_pe chunks per thread and step");
  __shared__ __attribute__((aligned(16))) T sC[KB * CP * 8];
  __shared__ __attribute__((aligned(16))) T sK[KB * KP * 8];
  __shared__ __attribute__((aligned(16))) T sD0[NW * DSW], sD1[NW * DSW];

  const T* __restrict__ kpe = (const T*)P.k_pe;
  const T* __restrict__ ds = (const T*)P.ds;
  const int S = P.S, H = P.H, TT = P.ds_T;

  int bh, qblk;
  ordered_block(P.order, blockIdx.x, bh, qblk);
  qblk = P.n_blocks - 1 - qblk;
  const int b = bh / H, h = bh % H;

  const int tid = threadIdx.x, l = tid & 63, n = l & 31, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & (NW - 1);
  const int t0 = (qblk * NW + wave) * TPW;  // this wave's query tiles t0 .. t0 + TPW - 1
  int nk[TPW];
  const T* dtile[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const bool ok = t0 + i < TT;
    nk[i] = ok ? ds_tile_keys(TT, P.causal, t0 + i) : 0;  // keys stored for the tile
    dtile[i] = ds + (ok ? ds_tile_offset(TT, P.causal, bh, t0 + i) : 0);
  }
  const int kend = P.causal ? min(S, (qblk + 1) * NW * TPW * 32) : S;
  const int nsteps = (kend + KB - 1) / KB;

  // W_h^T rows of this wave's column block in the order pi (bits 2 and 3 swapped), so
  // that lane (n, g) of the rebuild accumulator holds columns 16 hh + 8 g + e (the
  // fragment-ordered copy of W^T holds them so)
  frag_t<T> wf[NKS];
  {
    // W_h^T in fragment order: fragment (column block wave, step ks) at wt + ks * 512
    const T* wt = (const T*)P.w_t + ((size_t)h * (DKVH / 32) + wave) * NKS * 512 + l * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) wf[ks] = *reinterpret_cast<const frag_t<T>*>(wt + ks * 512);
  }
  const T* cg = (const T*)P.c_kv + (size_t)b * S * DC;

  f32x16 dqa[TPW][DQK / 32];
#pragma unroll
  for (int i = 0; i < TPW; ++i)
#pragma unroll
    for (int j = 0; j < DQK / 32; ++j) dqa[i][j] = f32x16{};

  // copies of step s: latent rows kt .. kt + 63 (rows past S clamped: their dS is zero),
  // wave w rows 16 w ..; the wave's dS^T blocks (a dummy block when not stored); k_pe rows
  // through registers (stored into the K tile after the next barrier)
  auto load_latent = [&](int kt) {
#pragma unroll
    for (int i = 0; i < KB / NW; ++i) {
      const int r = wave * (KB / NW) + i;
      g2lds16(cg + (size_t)min(kt + r, S - 1) * DC + l * 8, sC + r * CP * 8);
    }
  };
  auto load_ds = [&](T* sD, int kt) {
#pragma unroll
    for (int i = 0; i < TPW; ++i)
#pragma unroll
      for (int sub = 0; sub < 2; ++sub) {
        const int kb = kt + 32 * sub;
        const T* src = kb < nk[i] ? dtile[i] + (size_t)kb * 32 : dtile[i];
        T* dst = sD + wave * DSW + (i * 2 + sub) * 1024;
        g2lds16(src + l * 8, dst);
        g2lds16(src + 512 + l * 8, dst + 512);
      }
  };
  chunk16 pe[2];
  auto load_pe = [&](int kt) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = tid + i * 64 * NW, r = c / (DR / 8), ch = c % (DR / 8);
      pe[i] = *reinterpret_cast<const chunk16*>(kpe + (size_t)(b * S + min(kt + r, S - 1)) * DR + ch * 8);
    }
  };
  auto store_pe = [&]() {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = tid + i * 64 * NW, r = c / (DR / 8), ch = c % (DR / 8);
      *reinterpret_cast<chunk16*>(sK + r * KP * 8 + DN + ch * 8) = pe[i];
    }
  };

  constexpr int PF = 3;
  load_latent(0);
  load_ds(sD0, 0);
  load_pe(0);
  auto step = [&](auto stage, int st) {
    constexpr int SD = decltype(stage)::value;
    T* sDc = SD == 0 ? sD0 : sD1;  // this step's dS^T stage
    T* sDn = SD == 0 ? sD1 : sD0;  // the next step's
    const int kt = st * KB;
    wait_vmem();      // this wave's copies of step st (latent rows, dS^T, k_pe) have landed
    __syncthreads();  // everyone's; the previous step's reads of sK and of sDn are done
    store_pe();
    {  // K_nope column block `wave` for keys kt .. kt + 63: two chains, one per 32-key half
      auto c_frag = [&](int i) {  // product i: contraction step i / 2 of key half i % 2
        return *reinterpret_cast<const frag_t<T>*>(sC + (32 * (i & 1) + n) * CP * 8 + (i >> 1) * 16 + 8 * g);
      };
      f32x16 acc[2] = {f32x16{}, f32x16{}};
      frag_t<T> cb[PF + 1];
#pragma unroll
      for (int i = 0; i < PF; ++i) cb[i] = c_frag(i);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 2 * NKS; ++i) {
        if (i + PF < 2 * NKS) cb[(i + PF) % (PF + 1)] = c_frag(i + PF);
        mma(acc[i & 1], wf[i >> 1], cb[i % (PF + 1)]);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int kh = 0; kh < 2; ++kh) {
        T* dst = sK + (32 * kh + n) * KP * 8 + wave * 32 + 8 * g;
        *reinterpret_cast<bf16x8*>(dst) = acc_to_frag<T>(acc[kh], 0);
        *reinterpret_cast<bf16x8*>(dst + 16) = acc_to_frag<T>(acc[kh], 1);
      }
    }
    __syncthreads();  // the whole K tile is in LDS; every wave's reads of sC are done
    if (st + 1 < nsteps) {  // the next step's copies, behind this step's dQ products
      load_latent(kt + KB);
      load_ds(sDn, kt + KB);
      load_pe(kt + KB);
    }
#pragma unroll
    for (int sub = 0; sub < 2; ++sub) {
      const T* tk = sK + 32 * sub * KP * 8;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const int ra = kk * 16 + 4 * g;
        bf16x8 zf[TPW];
#pragma unroll
        for (int i = 0; i < TPW; ++i) zf[i] = pad_tr_frag<4>(sDc + wave * DSW + (i * 2 + sub) * 1024, ra, ra + 8, 0);
#pragma unroll
        for (int db = 0; db < DQK / 32; ++db) {
          const bf16x8 kf = pad_tr_frag<KP>(tk, ra, ra + 8, db * 32);
          // wave-uniform: key blocks past a tile's queries hold no dS for it
#pragma unroll
          for (int i = 0; i < TPW; ++i)
            if (kt + 32 * sub < nk[i]) mma(dqa[i][db], kf, zf[i]);
        }
      }
    }
  };
  for (int st = 0; st < nsteps; st += 2) {
    step(std::integral_constant<int, 0>{}, st);
    if (st + 1 < nsteps) step(std::integral_constant<int, 1>{}, st + 1);
  }

#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const int my_q = (t0 + i) * 32 + ds_query_of_position(n);
    if (t0 + i >= TT || my_q >= S) continue;
    T* dqr = (T*)P.dq + ((size_t)(b * S + my_q) * H + h) * DQK;
#pragma unroll
    for (int db = 0; db < DQK / 32; ++db)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = to_elem<T>(dqa[i][db][4 * rr + e] * P.scale);
        *reinterpret_cast<bf16x4*>(dqr + db * 32 + rr * 8 + g * 4) = v;
      }
  }
}

}  // namespace

// dq_ds_kernel's shapes: 8 waves (two per SIMD, which hides the latency of the dS^T stream and
// shares each K block among 256 queries), or 4 when 8 would give at most this many workgroups
// (then the longest chain of key blocks bounds it, and that runs faster alone on its SIMD).
// Both give the same bits. Measured (us, 8 / 4 waves; 8-wave workgroups): 2048 tokens x 16
// heads 42 / 30 (128), 2048 x 32 47 / 41 (256), 4096 x 16 90 / 71 (256), 8192 x 16 243 / 271
// (512), 2 x 5001 x 16 204 / 221 (640).
constexpr long long kDqNarrowMaxGroups = 320;

// dq_rec_kernel's shape: 4 waves (one per SIMD, 128 queries per workgroup). Measured at
// S=16384, H=16: 2.16-2.38 ms; 8 waves need more than their 256 registers (98 spilled):
// 7.8 ms. Interleaving one key block's dS arithmetic with the other's MFMAs in a pinned
// order measured 2 % slower than the plain order.
#ifndef DQ_REC_WAVES
#define DQ_REC_WAVES 4
#endif

template <typename T, int DN, int DR, int DV>
hipError_t launch_bwd_dq(bwd::BwdParams P, int B, hipStream_t st) {
  if constexpr (sizeof(T) == 2 && DN + DR == 192 && DV == 128) {
    if (P.ds) {
      if (P.w_t && P.d_c == kFusedMaxDc) {
        constexpr int TPW = 2;
        P.n_blocks = (P.ds_T + 4 * TPW - 1) / (4 * TPW);
        const dim3 grid = order_grid(P, B);
        dq_ds_fused2_kernel<DN, DR, DV, kFusedMaxDc, TPW><<<grid, 256, 0, st>>>(P);
      } else if (P.w_t) {
        constexpr int WPH = 8;
        P.n_blocks = (P.ds_T + WPH - 1) / WPH;
        const dim3 grid = order_grid(P, B);
        dq_ds_fused_kernel<DN, DR, DV><<<grid, 64 * WPH, 0, st>>>(P);
      } else {
        const int nb8 = (P.ds_T + 7) / 8;
        if ((long long)nb8 * P.H * B > kDqNarrowMaxGroups) {
          P.n_blocks = nb8;
          const dim3 grid = order_grid(P, B);
          dq_ds_kernel<DN, DR, DV, 8><<<grid, 512, 0, st>>>(P);
        } else {
          P.n_blocks = (P.ds_T + 3) / 4;
          const dim3 grid = order_grid(P, B);
          dq_ds_kernel<DN, DR, DV, 4><<<grid, 256, 0, st>>>(P);
        }
      }
      return hipGetLastError();
    }
  }
  if constexpr (sizeof(T) == 2 && DN >= 64) {
    // no dS^T store: recompute S, P, dP and dS per key tile
    constexpr int RW = DQ_REC_WAVES;
    P.n_blocks = (P.S + 32 * RW - 1) / (32 * RW);
    const dim3 grid = order_grid(P, B);
    dq_rec_kernel<DN, DR, DV, RW><<<grid, 64 * RW, 0, st>>>(P);
  } else {
    P.n_blocks = (P.S + 63) / 64;
    const dim3 grid = order_grid(P, B);
    dq_kernel<T, DN, DR, DV><<<grid, 256, 0, st>>>(P);
  }
  return hipGetLastError();
}

#define LAGA_INST_DQ(T, DN, DR, DV) template hipError_t launch_bwd_dq<T, DN, DR, DV>(bwd::BwdParams, int, hipStream_t);
#ifndef LAGA_HALF_WIDTHS
LAGA_INST_DQ(bf16, 128, 64, 128)
LAGA_INST_DQ(float, 128, 64, 128)
LAGA_INST_DQ(bf16, 32, 16, 32)
LAGA_INST_DQ(float, 32, 16, 32)
#else
LAGA_INST_DQ(bf16, 64, 32, 64)
LAGA_INST_DQ(float, 64, 32, 64)
#endif

}  // namespace laga
