// dc_kv and dW of a small problem in one launch: gemm.hip's ring tiles as a function.
#define LAGA_GEMM_PAIR
#include "gemm.hip"

namespace laga {

namespace {

// dc and dW in one launch (128 x 128 tiles, workgroups [0, n_dc) and the rest), for problems
// whose tiles of both fit the chip at once: alone, neither fills it.
__global__ __launch_bounds__(256, 2) void gemm_dc_dw_kernel(GemmPairArgs a) {
  __shared__ __attribute__((aligned(16))) bf16 sm[3 * ring_stage(128, 128, 1)];
  const int id = blockIdx.x;
  if (id < a.n_dc)
    gemm_ring_tile<128, 128, 4, 2, 3, false, false, 1, float>(sm, id % a.tiles_dc, id / a.tiles_dc, a.dkv, a.w,
                                                              a.dkv_lo, a.dc, a.tokens, a.d_c, a.ncol, a.ncol, a.ncol,
                                                              a.d_c, a.chunk_dc, (long long)a.tokens * a.d_c);
  else
    gemm_ring_tile<128, 128, 4, 2, 3, true, true, 2, float>(sm, (id - a.n_dc) % a.tiles_dw, (id - a.n_dc) / a.tiles_dw,
                                                            a.c, a.dkv, a.dkv_lo, a.dw, a.d_c, a.ncol, a.tokens, a.d_c,
                                                            a.ncol, a.ncol, a.chunk_dw, (long long)a.d_c * a.ncol);
}

}  // namespace

void launch_gemm_pair(const GemmPairArgs& a, int groups, hipStream_t st) {
  gemm_dc_dw_kernel<<<groups, 256, 0, st>>>(a);
}

}  // namespace laga
