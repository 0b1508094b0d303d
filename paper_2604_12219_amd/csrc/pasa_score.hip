// Stage 1 of the PASA forward on gfx950: block-pooled routing logits (pasa_score.hpp).
#include "pasa_score.hpp"

namespace {

template <int D>
__global__ void __launch_bounds__(256) pool_mean_kernel(ScoreParams p) {
  __shared__ __attribute__((aligned(16))) char lds[kPoolLds];
  pool_mean<D>(p, blockIdx.x, blockIdx.y, blockIdx.z, lds);
}

template <int D>
__global__ void __launch_bounds__(256) score_gemm_kernel(ScoreParams p, int runs) {
  __shared__ __attribute__((aligned(16))) char lds[kScoreLds];
  score_gemm<D>(p, runs, blockIdx.x, lds);
}

template <int D>
hipError_t launch(const ScoreParams& p, hipStream_t stream) {
  const dim3 gp(p.nb, p.bh, p.pool_k ? 2 : 1);  // z = 0 pools the queries, z = 1 the keys
  hipLaunchKernelGGL(pool_mean_kernel<D>, gp, dim3(256), 0, stream, p);
  int runs;
  const dim3 gg(score_workgroups(p, &runs));
  hipLaunchKernelGGL(score_gemm_kernel<D>, gg, dim3(256), 0, stream, p, runs);
  return hipGetLastError();
}

}  // namespace

hipError_t pasa_launch_block_score(const ScoreParams& p, hipStream_t stream) {
  return p.d == 128 ? launch<128>(p, stream) : launch<64>(p, stream);
}
