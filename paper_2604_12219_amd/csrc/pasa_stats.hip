// Key/value block statistics of the PASA forward (pasa_stats.hpp) by themselves, and the covariance-aware routing prior.
#include "pasa_stats.hpp"

namespace {

template <int D>
__global__ void __launch_bounds__(256, 2) kv_stats_kernel(StatsParams p) {
  __shared__ __attribute__((aligned(16))) char smem[2 * 64 * 2 * D];
  kv_stats<D>(p, blockIdx.x, blockIdx.y, smem);
}

template <int D>
__global__ void __launch_bounds__(256) hg_finish_kernel(StatsParams p) {
  __shared__ __attribute__((aligned(16))) char lds[kFinishLds];
  hg_finish<D>(p, blockIdx.x, blockIdx.y, blockIdx.z, lds);
}

// Covariance-aware routing prior (Eq.8): beta_j = log(|| H_j - Hg_{g(j)} ||_F + eps) for every key block.
// The same sweep as kv_stats_kernel, but H_j is formed per block and compared, element by element in fp32, with the
// group mean, from the group's sum that the statistics left.
// Nothing but beta is written.
template <int D>
__global__ void __launch_bounds__(256) key_prior_kernel(StatsParams p, float eps, float* beta) {
  constexpr int TI = D / 64;
  constexpr int TILE_BYTES = 64 * 2 * D;
  __shared__ __attribute__((aligned(16))) char smem[2 * TILE_BYTES];
  __shared__ float red_s[2][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5;
  const int u = blockIdx.x, bh = blockIdx.y;
  const int j_lo = u * p.prior_unit, j_hi = min(j_lo + p.prior_unit, p.nb);
  const int tin0 = (wave >> 1) * TI, tout0 = (wave & 1) * TI;

  // the group these blocks belong to, and its mean
  const int g = j_lo / p.group;
  const float inv_blocks = 1.0f / (float)(min((g + 1) * p.group, p.nb) - g * p.group);
  const float* const group_sum = p.group_sum + ((int64_t)bh * p.sum_head + (int64_t)g * p.sum_group) * D * D;
  f32x16 mean[TI][TI];
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TI; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        mean[a][b][r] = group_sum[(32 * (tin0 + a) + mfma_row(r, h)) * D + 32 * (tout0 + b) + (lane & 31)] * inv_blocks;

  f32x16 acc[TI][TI];
#pragma unroll
  for (int a = 0; a < TI; ++a)
#pragma unroll
    for (int b = 0; b < TI; ++b) acc[a][b] = f32x16{0};

  int parity = 0;  // red_s is double-buffered: one barrier per block is enough
  sweep_unit<D>(p, bh, j_lo, j_hi, smem, smem + TILE_BYTES, acc,
                [&](int j, int len, f32x16 (&acc)[TI][TI], const f32x16 (&ksum)[TI], const f32x16 (&vsum)[TI]) {
    const float inv_len = 1.0f / (float)len;
    float ss = 0.f;
#pragma unroll
    for (int a = 0; a < TI; ++a)
#pragma unroll
      for (int b = 0; b < TI; ++b) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float hj = acc[a][b][r] - ksum[a][r] * inv_len * vsum[b][0];
          const float dlt = hj - mean[a][b][r];
          ss = fmaf(dlt, dlt, ss);
        }
        acc[a][b] = f32x16{0};
      }
#pragma unroll
    for (int sh = 32; sh >= 1; sh >>= 1) ss += __shfl_xor(ss, sh);
    if (lane == 0) red_s[parity][wave] = ss;
    __syncthreads();
    if (tid == 0)
      beta[(int64_t)bh * p.nb + j] = logf(sqrtf(red_s[parity][0] + red_s[parity][1] + red_s[parity][2] + red_s[parity][3]) + eps);
    parity ^= 1;  // the other half is next written after the sweep's own barrier and this one
  });
}

template <int D>
hipError_t launch(const StatsParams& p, hipStream_t stream) {
  hipLaunchKernelGGL(kv_stats_kernel<D>, dim3(stats_workgroups(p), p.bh), dim3(256), 0, stream, p);
  if (finish_pieces(p)) hipLaunchKernelGGL(hg_finish_kernel<D>, dim3(p.n_groups, p.bh, finish_pieces(p)), dim3(256), 0, stream, p);
  return hipGetLastError();
}

}  // namespace

hipError_t pasa_launch_kv_stats(const StatsParams& p, hipStream_t stream) {
  return p.d == 128 ? launch<128>(p, stream) : launch<64>(p, stream);
}

hipError_t pasa_launch_key_prior(const StatsParams& p, float eps, float* beta, hipStream_t stream) {
  dim3 g1((p.nb + p.prior_unit - 1) / p.prior_unit, p.bh);
  if (p.d == 128) hipLaunchKernelGGL(key_prior_kernel<128>, g1, dim3(256), 0, stream, p, eps, beta);
  else hipLaunchKernelGGL(key_prior_kernel<64>, g1, dim3(256), 0, stream, p, eps, beta);
  return hipGetLastError();
}
