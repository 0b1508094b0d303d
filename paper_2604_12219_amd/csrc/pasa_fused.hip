// Statistics and scoring in the same launches, for the calls that run both (the whole forward): neither needs the other's first kernel.
// A launch with the gap before it takes 2.5 us or more whatever is in it, and the statistics' few workgroups leave most of the device idle for as long as
// they walk their units: the pooling fills it.  us, four launches / two (with the keys pooled): 1024 tokens, 2 heads, d = 64 12.1 / 7.6;
// 4140 tokens, 4 heads, d = 128, groups of 64 22.6 / 16.0.  Which calls take it: stats_and_score_together in pasa_api.hip.
#include "pasa_score.hpp"
#include "pasa_stats.hpp"

namespace {

// kv_stats of every unit, then pool_mean of every block (the units take longest, so they come first)
template <int D>
__global__ void __launch_bounds__(256, 2) stats_pool_kernel(StatsParams t, ScoreParams p) {
  __shared__ __attribute__((aligned(16))) char smem[2 * 64 * 2 * D];
  static_assert(sizeof(smem) >= kPoolLds, "");
  const int n_stats = t.bh * t.n_units, e = (int)blockIdx.x - n_stats;
  if (e < 0) {
    kv_stats<D>(t, blockIdx.x % t.n_units, blockIdx.x / t.n_units, smem);
  } else {
    const int row = e / p.nb;
    pool_mean<D>(p, e % p.nb, row % p.bh, row / p.bh, smem);
  }
}

// score_gemm and hg_finish; `pieces` of the latter per head and group
template <int D>
__global__ void __launch_bounds__(256) score_finish_kernel(ScoreParams p, int runs, int n_score, StatsParams t, int pieces) {
  __shared__ __attribute__((aligned(16))) char lds[kScoreLds];
  static_assert(sizeof(lds) >= kFinishLds, "");
  const int e = (int)blockIdx.x - n_score;
  if (e < 0) score_gemm<D>(p, runs, blockIdx.x, lds);
  else hg_finish<D>(t, (e / pieces) % t.n_groups, e / (pieces * t.n_groups), e % pieces, lds);
}

template <int D>
hipError_t launch(const StatsParams& t, const ScoreParams& p, hipStream_t stream) {
  hipLaunchKernelGGL(stats_pool_kernel<D>, dim3(t.bh * (t.n_units + p.nb * (p.pool_k ? 2 : 1))), dim3(256), 0, stream, t, p);
  int runs;
  const int n_score = (int)score_workgroups(p, &runs), pieces = (int)finish_pieces(t);
  hipLaunchKernelGGL(score_finish_kernel<D>, dim3(n_score + t.bh * t.n_groups * pieces), dim3(256), 0, stream, p, runs, n_score, t, pieces > 0 ? pieces : 1);
  return hipGetLastError();
}

}  // namespace

hipError_t pasa_launch_stats_and_score(const StatsParams& t, const ScoreParams& p, hipStream_t stream) {
  return t.d == 128 ? launch<128>(t, p, stream) : launch<64>(t, p, stream);
}
