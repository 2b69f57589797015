// Generic key-stationary dK / dV kernel of the attention backward (fp32 at every head width,
// and bf16 at 32/16/32-wide heads). Its own source file because it is compiled with the MFMA
// results in VGPRs (no AGPR<->VGPR copies around the softmax arithmetic on the
// accumulators), a choice that makes the tuned bf16 kernel of attn_bwd.hip spill.
//
// P = softmax(scale * Q K^T) is recomputed from the saved row log-sum-exp; per key
// block: dV = P^T dO, dP = dO V^T, dZ = P * (dP - delta), dK = scale dZ^T Q (the
// key-side half of the backward; dQ is the query-stationary pass of attn_bwd_dq.hip).
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

// ------------------------------------------------------------------ dK, dV
// A workgroup of four waves owns 64 keys of one head: waves 0, 1 take the even 32-query tiles,
// waves 2, 3 the odd ones of the same keys (32 per wave; K, V and the dK^T / dV^T
// accumulators in registers), and the two partial sums meet in LDS at the end. The work on a
// tile has two equal halves - A: S = Q K^T, dP = dO V^T and the softmax, C: dV^T += dO^T P,
// dK^T += Q^T dZ - and phase p runs A of tile p on one pair of waves beside C of tile p - 1 on
// the other, so a tile is needed for two phases and three LDS slots do (fp32 tiles of 192/128
// wide heads are 43 KB: a slot more would not fit): one with this phase's, one with the last
// one's, one being filled for the next by direct global->LDS copies.
// Bound: fp32 MFMA (2048 tokens, 16 heads, 192/128-wide: 280 us of products at the peak rate).
// The first keys see every query, so their chain of tiles is the kernel's time when there
// are no more workgroups than CUs; two pairs of waves halve it. Before (128 keys per workgroup,
// each wave on every tile) / now, us, fp32: 2048 tokens, 16 heads 786 / 390, 32 heads x 4000 3100 / 2730;
// 256 tokens, 4 heads of 48/32 51 / 22; bf16, 1000 tokens, 16 heads of 48/32 120 / 40.
template <typename T, int DN, int DR, int DV>
__global__ __launch_bounds__(256, DN == 128 ? 1 : 2) void dkdv_kernel(BwdParams P) {
  constexpr int DQK = DN + DR, DKVH = DN + DV, DQK32 = round32(DQK), NDK = DQK32 / 32, NDV = DV / 32;
  constexpr int BQ = 32, BK = 64, NS = 3, E = Elems16<T>::n;
  constexpr int PQ = lds_pitch<T>(DQK32), PO = lds_pitch<T>(DV);
  constexpr int QCH = DQK / E, OCH = DV / E;  // chunks per row
  static_assert(QCH <= 64 && OCH <= 64, "one copy instruction per row");
  constexpr int TQ = BQ * PQ, TO = BQ * PO;
  __shared__ __attribute__((aligned(16))) T sm[NS * (TQ + TO)];  // Q slots, then dO slots
  T* const sOm = sm + NS * TQ;
  __shared__ __attribute__((aligned(16))) float sLD[NS][2 * BQ];

  const T* __restrict__ q = (const T*)P.q;
  const T* __restrict__ kpe = (const T*)P.k_pe;
  const T* __restrict__ kv = (const T*)P.kv;
  const T* __restrict__ dout = (const T*)P.dout;
  const int S = P.S, H = P.H;

  int bh, kb;  // the first key blocks see the most queries
  ordered_block(P.order, blockIdx.x, bh, kb);
  const int b = bh / H, h = bh % H;

  const int tid = threadIdx.x, l = tid & 63, n = l & 31, g = l >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
  const int kw = wave & 1, qw = wave >> 1;
  const int k0 = kb * BK + kw * 32;  // first key of this wave
  const int my_k = k0 + n;

  // zero the padding columns [DQK, DQK32) of every slot once: transposing reads of Q^T
  // blocks touch them
  if (DQK32 > DQK)
    for (int i = tid; i < NS * BQ * (DQK32 - DQK); i += 256) {
      const int st = i / (BQ * (DQK32 - DQK)), j = i % (BQ * (DQK32 - DQK));
      sm[st * TQ + (j / (DQK32 - DQK)) * PQ + DQK + j % (DQK32 - DQK)] = to_elem<T>(0.f);
    }

  // this lane's key and value rows (B operands of S = Q K^T and dP = dO V^T)
  frag_t<T> kf[DQK / 16], vf[DV / 16];
  {
    const bool ok = my_k < S;
    const size_t row = (size_t)(b * S + (ok ? my_k : 0));
    const T* kvr = kv + (row * H + h) * DKVH;
#pragma unroll
    for (int ks = 0; ks < DQK / 16; ++ks) {
      const T* src = ks < DN / 16 ? kvr + ks * 16 + 8 * g : kpe + row * DR + (ks - DN / 16) * 16 + 8 * g;
      if (ok) kf[ks] = *reinterpret_cast<const frag_t<T>*>(src);
      else
#pragma unroll
        for (int e = 0; e < 8; ++e) kf[ks][e] = to_elem<T>(0.f);
    }
#pragma unroll
    for (int ks = 0; ks < DV / 16; ++ks) {
      if (ok) vf[ks] = *reinterpret_cast<const frag_t<T>*>(kvr + DN + ks * 16 + 8 * g);
      else
#pragma unroll
        for (int e = 0; e < 8; ++e) vf[ks][e] = to_elem<T>(0.f);
    }
  }

  f32x16 dk[NDK], dv[NDV];
#pragma unroll
  for (int i = 0; i < NDK; ++i) dk[i] = f32x16{};
#pragma unroll
  for (int i = 0; i < NDV; ++i) dv[i] = f32x16{};

  const int qt_begin = P.causal ? kb * BK : 0;
  const int nt = (S - qt_begin + BQ - 1) / BQ;
  // Slot <- tile j: wave w copies rows 8 w .. of Q and of dO, one instruction per row (lane l
  // chunk l); rows past S copy row S - 1 (masked below). lse2 and delta rows are padded to S_pad
  // (a multiple of 64 >= S): their BQ entries are copied whole by the last wave.
  const size_t hrow0 = (size_t)(b * S) * H + h, ld_row = (size_t)bh * P.S_pad;
  auto fill = [&](int st, int j) {
    const int qt = qt_begin + j * BQ;
    if (l < QCH)
#pragma unroll
      for (int i = 0; i < BQ / 4; ++i) {
        const int r = wave * (BQ / 4) + i;
        g2lds16_so(q + (hrow0 + (size_t)min(qt + r, S - 1) * H) * DQK, 16u * l, sm + st * TQ + r * PQ);
      }
    if (l < OCH)
#pragma unroll
      for (int i = 0; i < BQ / 4; ++i) {
        const int r = wave * (BQ / 4) + i;
        g2lds16_so(dout + (hrow0 + (size_t)min(qt + r, S - 1) * H) * DV, 16u * l, sOm + st * TO + r * PO);
      }
    if (wave == 3 && l < BQ / 2) {
      const float* src = l < BQ / 4 ? P.lse2 + ld_row + qt + 4 * l : P.delta + ld_row + qt + 4 * (l - BQ / 4);
      g2lds16(src, &sLD[st][0]);
    }
  };

  // A of tile j (slot st): P in sa and dZ in dp, rows = queries (r/4)*8 + g*4 + r%4, column = my key
  f32x16 sa, dp;
  auto half_a = [&](int st, int j) {
    const T *sQ = sm + st * TQ, *sO = sOm + st * TO;
    const float *sL = sLD[st], *sD = sLD[st] + BQ;
    const int qt = qt_begin + j * BQ;
    sa = f32x16{};
    dp = f32x16{};
#pragma unroll
    for (int ks = 0; ks < DQK / 16; ++ks) mma(sa, lds_frag<T>(sQ + n * PQ + ks * 16 + 8 * g), kf[ks]);
#pragma unroll
    for (int ks = 0; ks < DV / 16; ++ks) mma(dp, lds_frag<T>(sO + n * PO + ks * 16 + 8 * g), vf[ks]);
    const bool need_mask = (P.causal && qt < k0 + 31) || (qt + BQ > S);
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int qrow = rr * 8 + g * 4;
      const f32x4 lq = *reinterpret_cast<const f32x4*>(sL + qrow);
      const f32x4 dq = *reinterpret_cast<const f32x4*>(sD + qrow);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = rr * 4 + e;
        float p = fast_exp2(sa[r] * P.scale_log2 - lq[e]);
        if (need_mask) {
          const int qi = qt + qrow + e;
          if (qi >= S || (P.causal && my_k > qi)) p = 0.f;
        }
        sa[r] = p;
        dp[r] = p * (dp[r] - dq[e]);
      }
    }
  };
  auto half_c = [&](int st) {
    const T *sQ = sm + st * TQ, *sO = sOm + st * TO;
#pragma unroll
    for (int kk = 0; kk < BQ / 16; ++kk) {
      const frag_t<T> pf = acc_to_frag<T>(sa, kk), zf = acc_to_frag<T>(dp, kk);
      const int ra = kk * 16 + 4 * g;
#pragma unroll
      for (int db = 0; db < NDV; ++db) mma(dv[db], TrRead<T>::get(sO, PO, ra, ra + 8, db * 32), pf);
#pragma unroll
      for (int db = 0; db < NDK; ++db) mma(dk[db], TrRead<T>::get(sQ, PQ, ra, ra + 8, db * 32), zf);
    }
  };
  // tiles that this wave works on at all (wave-uniform): its keys exist and some query sees them
  auto active = [&](int j) { return k0 < S && (!P.causal || qt_begin + j * BQ + BQ - 1 >= k0); };

  // start of phase p: tile p is there, tile p + 1 on its way into the slot of tile p - 2
  auto phase = [&](int p) {
    wait_vmem();      // this wave's copies of tile p have landed
    __syncthreads();  // everyone's; tile p - 2 is no longer read
    if (p + 1 < nt) fill((p + 1) % NS, p + 1);
  };
  fill(0, 0);
  if (qw) phase(0);
  for (int p = qw; p < nt; p += 2) {
    const bool on = active(p);
    phase(p);
    if (on) half_a(p % NS, p);
    phase(p + 1);
    if (on) half_c(p % NS);
  }
  if ((nt & 1) == qw) phase(nt);  // every wave goes through phases 0 .. nt

  // the first wave of a pair takes the other's dK and finishes it, the second the first's dV
  // (even + odd tiles)
  __syncthreads();
  static_assert(2 * (NDK + NDV) * 4096 <= (int)sizeof(T) * NS * (TQ + TO), "partials fit the slots");
  // dK partials of both key halves, then dV's, 4 KB per 32 x 32 block
  auto block = [&](int i) { return (float*)sm + i * 1024; };
  auto put_x = [&](int i, const f32x16& a) {
    float* x = block(i) + l * 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) *reinterpret_cast<f32x4*>(x + r * 256) = f32x4{a[4 * r], a[4 * r + 1], a[4 * r + 2], a[4 * r + 3]};
  };
  auto add_x = [&](int i, f32x16& a) {
    const float* x = block(i) + l * 4;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(x + r * 256);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[4 * r + e] += v[e];
    }
  };
  if (qw == 0) {
#pragma unroll
    for (int i = 0; i < NDV; ++i) put_x(2 * NDK + kw * NDV + i, dv[i]);
  } else {
#pragma unroll
    for (int i = 0; i < NDK; ++i) put_x(kw * NDK + i, dk[i]);
  }
  __syncthreads();
  if (qw == 0) {
#pragma unroll
    for (int i = 0; i < NDK; ++i) add_x(kw * NDK + i, dk[i]);
  } else {
#pragma unroll
    for (int i = 0; i < NDV; ++i) add_x(2 * NDK + kw * NDV + i, dv[i]);
  }

  if (my_k >= S) return;
  const size_t row = (size_t)(b * S + my_k) * H + h;
  T* dkvr = (T*)P.dkv + row * DKVH;
  T* dkvl = (T*)P.dkv_lo + row * DKVH;
  float* dper = P.dkpe_h + row * DR;
  // dKV as hi (+ lo for bf16): lo = bf16(x - hi) carries the next 8 bits for the GEMMs
  auto put4 = [&](int col, float a0, float a1, float a2, float a3) {
    typename FragOf<T>::half hi = {to_elem<T>(a0), to_elem<T>(a1), to_elem<T>(a2), to_elem<T>(a3)};
    *reinterpret_cast<typename FragOf<T>::half*>(dkvr + col) = hi;
    if (sizeof(T) == 2) {
      typename FragOf<T>::half lo = {to_elem<T>(a0 - to_f32(hi[0])), to_elem<T>(a1 - to_f32(hi[1])),
                                     to_elem<T>(a2 - to_f32(hi[2])), to_elem<T>(a3 - to_f32(hi[3]))};
      *reinterpret_cast<typename FragOf<T>::half*>(dkvl + col) = lo;
    }
  };
  if (qw == 0) {
#pragma unroll
    for (int db = 0; db < NDK; ++db)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr) {
        const int d = db * 32 + rr * 8 + g * 4;
        const float a0 = dk[db][4 * rr] * P.scale, a1 = dk[db][4 * rr + 1] * P.scale;
        const float a2 = dk[db][4 * rr + 2] * P.scale, a3 = dk[db][4 * rr + 3] * P.scale;
        if (d < DN) {
          put4(d, a0, a1, a2, a3);
        } else if (d < DQK) {
          f32x4 v = {a0, a1, a2, a3};
          *reinterpret_cast<f32x4*>(dper + (d - DN)) = v;
        }
      }
  } else {
#pragma unroll
    for (int db = 0; db < NDV; ++db)
#pragma unroll
      for (int rr = 0; rr < 4; ++rr)
        put4(DN + db * 32 + rr * 8 + g * 4, dv[db][4 * rr], dv[db][4 * rr + 1], dv[db][4 * rr + 2], dv[db][4 * rr + 3]);
  }
}

}  // namespace

template <typename T, int DN, int DR, int DV>
hipError_t launch_dkdv_generic(BwdParams P, int B, hipStream_t st) {
  P.n_blocks = (P.S + 63) / 64;
  const dim3 grid = order_grid(P, B);
  dkdv_kernel<T, DN, DR, DV><<<grid, 256, 0, st>>>(P);
  return hipGetLastError();
}

#define LAGA_INST_DKDV(T, DN, DR, DV) \
  template hipError_t launch_dkdv_generic<T, DN, DR, DV>(BwdParams, int, hipStream_t);
LAGA_INST_DKDV(float, 128, 64, 128)  // bf16 at these widths runs dkdv32_kernel, at 64/32/64 dkdv_half_kernel
LAGA_INST_DKDV(bf16, 32, 16, 32)
LAGA_INST_DKDV(float, 32, 16, 32)
LAGA_INST_DKDV(float, 64, 32, 64)

}  // namespace laga
