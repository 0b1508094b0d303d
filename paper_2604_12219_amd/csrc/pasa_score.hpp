// Device side of stage 1 (block-pooled routing logits, Eq.8 without its softmax), by itself in pasa_score.hip and beside the statistics in
// pasa_fused.hip:
//   qbar_i = mean of the valid rows of query block i, kbar_j likewise          (HBM-bound reads)
//   scores[bh,i,j] = scale * qbar_i . kbar_j + key_bias[bh,j]                  (fp32 throughout)
#pragma once
#include "pasa_device.hpp"
#include "pasa_kernels.hpp"

namespace {

// One workgroup per (block, head, tensor): 16-byte loads along d, partial sums over rows in
// registers, a 16-way (or 32-way) reduction through LDS.
constexpr int kPoolLds = 8192;
template <int D>
PASA_DEVICE void pool_mean(const ScoreParams& p, int j, int bh, int which, char* lds) {
  constexpr int CPR = D / 8, RPP = 256 / CPR;  // 16-byte chunks per row, rows per pass
  static_assert(RPP * D * sizeof(float) == kPoolLds, "");
  float(*const part)[D] = reinterpret_cast<float(*)[D]>(lds);
  const int tid = threadIdx.x, c = tid % CPR, r = tid / CPR;
  const int64_t head_off = (int64_t)(bh / p.H) * p.stride_b + (int64_t)(bh % p.H) * p.stride_h;
  const uint16_t* src = (which ? p.k : p.q) + head_off;
  const int row0 = j * p.block, len = min(p.block, p.n - row0);
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int row = r; row < len; row += RPP) {
    const uint4 raw = *reinterpret_cast<const uint4*>(src + (int64_t)(row0 + row) * p.stride_n + c * 8);
    const uint32_t wds[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      acc[2 * e] += __uint_as_float(wds[e] << 16);
      acc[2 * e + 1] += __uint_as_float(wds[e] & 0xffff0000u);
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) part[r][c * 8 + e] = acc[e];
  __syncthreads();
  if (tid < D) {
    float s = 0.f;
#pragma unroll
    for (int rr = 0; rr < RPP; ++rr) s += part[rr][tid];
    // The mean leaves as two bf16 numbers, hi = bf16(mean) and lo = bf16(mean - hi) (together 16 significant bits),
    // so that the score kernel can multiply on the bf16 matrix cores.  Row layout: per quarter of 32 elements one
    // 128-byte line, 32 x hi then 32 x lo.
    const float mean = s / (float)len;
    const __bf16 hi = (__bf16)mean;
    const __bf16 lo = (__bf16)(mean - (float)hi);
    uint16_t* dst = reinterpret_cast<uint16_t*>((which ? p.kbar : p.qbar) + ((int64_t)bh * p.nb + j) * D);
    dst[(tid >> 5) * 64 + (tid & 31)] = __builtin_bit_cast(uint16_t, hi);
    dst[(tid >> 5) * 64 + 32 + (tid & 31)] = __builtin_bit_cast(uint16_t, lo);
  }
}

// scores: a workgroup of four waves computes 64x64 tiles, each wave a 32x32 quarter of a tile, on the bf16 matrix
// cores: with q = qh + ql and k = kh + kl (the split pooled means), q.k = qh.kh + qh.kl + ql.kh up to 2^-16 relative,
// accumulated in fp32 -- three bf16 MFMAs (32x32x16) instead of eight fp32 ones (32x32x2) per 16 elements of the
// contraction, five times less matrix time.  The pooled means are row-major, and an MFMA operand wants one ROW per
// lane, which as a global load would touch 64 cache lines per instruction.  So the contraction runs in quarters of
// 32 elements: a quarter of a row (hi and lo) is exactly one 128-byte line, the workgroup fetches the quarters of
// its 64 + 64 rows with fully coalesced 16-byte loads (eight lanes per line), parks them in LDS (rows padded to 144
// bytes: conflict-free 16-byte reads down a column of rows), and every lane reads its operands from there.  Two LDS
// buffers, one barrier a quarter.  What bounds a small grid is the time of a trip to memory: the quarters of a tile are requested all together (a quarter
// at a time, one ahead of the MFMAs, was a trip each), those of the next tile of the run during the last quarter's MFMAs, and the queries' stay in
// registers for the whole run.  With the runs of strips below, pooling and scores, us: 4140 tokens, 4 heads 8.9 -> 8.0; 32,760, 12 39.5 -> 38.4;
// 118,800, 3 56.3 -> 50.5; 75,600, 40 440 -> 415.  In a quarter, lane (x, h) holds elements [8h + 16m, 8h + 16m + 8) of its row for the MFMAs m = 0, 1.
constexpr int kScorePitch = 32 * 4 + 16, kScoreLds = 2 * 128 * kScorePitch;
template <int D>
PASA_DEVICE void score_gemm(const ScoreParams& p, int runs, int wg, char* lds_bytes) {
  constexpr int QF = 32;               // elements per quarter-row (stored as 32 bf16 hi + 32 bf16 lo = 32 floats' worth of bytes)
  constexpr int NQ = D / QF;           // quarters
  constexpr int PITCH = kScorePitch;   // bytes per LDS row
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, x = lane & 31, h = lane >> 5;
  // The hardware deals consecutive workgroup ids round-robin to the 8 XCDs: each XCD takes a run of consecutive strips, so that the pooled means of a
  // head are fetched into one L2 or two instead of eight.  (A head that is alone is fetched into all of them either way.  Strip by strip or column by column,
  // us: 230,000 tokens 42.8 / 42.1, 180,000 30.4 / 30.8, 262,144 49.1 / 46.9; 3 heads of 118,800 48.7 / 51.7)
  const int n_tiles = (p.nb + 63) / 64;
  const int per_head = runs * n_tiles, total = p.bh * per_head, per_xcd = (total + 7) / 8;
  const int slot = (wg & 7) * per_xcd + (wg >> 3);
  if (slot >= total) return;  // padding workgroup: leaves before any barrier
  const int bh = slot / per_head;
  const int within = slot % per_head;
  const int run_id = within % runs, i0 = (within / runs) * 64;
  // A workgroup owns a strip of 64 score rows and walks a run of 64-column tiles along it: the 256-byte row
  // segments of consecutive tiles are then written by the same compute unit one after the other, and the cache
  // lines that straddle two tiles (rows are not a multiple of a line long) are completed in its L2 instead of going
  // to memory as two partial lines from two different L2s (3x the bytes of the scores themselves when every tile
  // was a workgroup of its own).
  const int run = (n_tiles + runs - 1) / runs;
  const int jt0 = run_id * run, jt1 = min(jt0 + run, n_tiles);
  const float* const qbar = p.qbar + (int64_t)bh * p.nb * D;
  const float* const kbar = p.kbar + (int64_t)bh * p.nb * D;
  // loader role: thread t fetches 16-byte chunk (t & 7) of tile rows (t >> 3) + 32 i, i = 0..3 (rows 0..63 are
  // pooled queries, 64..127 pooled keys); rows past the end are clamped: their products are never stored
  const int ld_row = tid >> 3, ld_col = (tid & 7) * 4;
  typedef float f32x4 __attribute__((ext_vector_type(4)));  // (arrays of HIP's float4 were kept in scratch memory, four times the bytes of the scores)
  f32x4 sq[NQ][2], sk[NQ][2];
#pragma unroll
  for (int qtr = 0; qtr < NQ; ++qtr)
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      sq[qtr][i] = *reinterpret_cast<const f32x4*>(qbar + (int64_t)min(i0 + ld_row + 32 * i, p.nb - 1) * D + ld_col + qtr * QF);
      sk[qtr][i] = *reinterpret_cast<const f32x4*>(kbar + (int64_t)min(jt0 * 64 + ld_row + 32 * i, p.nb - 1) * D + ld_col + qtr * QF);
    }
  char* const park = lds_bytes + ld_row * PITCH + (tid & 7) * 16;
  // consumer role: wave (wi, wj) multiplies query rows 32 wi + x with key rows 32 wj + x
  const int a_off = (32 * (wave >> 1) + x) * PITCH + h * 16, b_off = (64 + 32 * (wave & 1) + x) * PITCH + h * 16;
#pragma unroll 1
  for (int jt = jt0; jt < jt1; ++jt) {
    const int j0 = jt * 64;
    f32x16 acc = {0};
#pragma unroll
    for (int qtr = 0; qtr < NQ; ++qtr) {
      // the buffer's readers finished before the previous barrier (NQ is even: a tile begins with the buffer that its predecessor did not end with)
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        *reinterpret_cast<f32x4*>(park + (qtr & 1) * 128 * PITCH + 32 * i * PITCH) = sq[qtr][i];
        *reinterpret_cast<f32x4*>(park + (qtr & 1) * 128 * PITCH + (64 + 32 * i) * PITCH) = sk[qtr][i];
      }
      __syncthreads();
      if (qtr + 1 == NQ && jt + 1 < jt1) {
#pragma unroll
        for (int n = 0; n < NQ; ++n)
#pragma unroll
          for (int i = 0; i < 2; ++i)
            sk[n][i] = *reinterpret_cast<const f32x4*>(kbar + (int64_t)min(j0 + 64 + ld_row + 32 * i, p.nb - 1) * D + ld_col + n * QF);
      }
      const char* buf = lds_bytes + (qtr & 1) * 128 * PITCH;
      // operand fragments of 8 bf16: [m] hi, [2 + m] lo of elements 8h + 16m .. + 8
      bf16x8 a[4], b[4];
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        a[c] = *reinterpret_cast<const bf16x8*>(buf + a_off + 64 * (c >> 1) + 32 * (c & 1));
        b[c] = *reinterpret_cast<const bf16x8*>(buf + b_off + 64 * (c >> 1) + 32 * (c & 1));
      }
#pragma unroll
      for (int m = 0; m < 2; ++m) {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[2 + m], b[m], acc, 0, 0, 0);  // ql kh  (small terms first)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m], b[2 + m], acc, 0, 0, 0);  // qh kl
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[m], b[m], acc, 0, 0, 0);      // qh kh
      }
    }
    // result register 4g + r of lane (x, h) is row 8g + 4h + r, column x of the wave's quarter
    const int j = j0 + 32 * (wave & 1) + x, i = 32 * (wave >> 1) + 4 * h;
    if (j < p.nb) {
      const float bias = p.key_bias ? p.key_bias[(int64_t)bh * p.nb + j] : 0.f;
      // A uniform row address and the lane's offset in the strip (64 rows: it fits 32 bits).  With an address a row the compiler kept the sixteen of them in
      // registers along the strip, 136 instead of 106, and three workgroups a compute unit instead of four: 1 head of 262,144 tokens 52.3 / 49.1 us
      float* const strip = p.scores + ((int64_t)bh * p.nb + i0) * p.nb;
      const uint32_t off = (uint32_t)i * (uint32_t)p.nb + (uint32_t)j;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + (r & 3);
        if (i0 + i + row < p.nb) (strip + (int64_t)row * p.nb)[off] = fmaf(acc[r], p.scale, bias);
      }
    }
  }
}

// Workgroups of score_gemm: strips of 64 rows; a strip is cut into runs of column tiles only as far as it takes to fill the device
inline unsigned score_workgroups(const ScoreParams& p, int* runs_out) {
  const int tiles = (p.nb + 63) / 64;
  const int64_t strips = (int64_t)tiles * p.bh;
  int runs = (int)((2048 + strips - 1) / strips);
  runs = runs < 1 ? 1 : runs > tiles ? tiles : runs;
  *runs_out = runs;
  return (unsigned)(8 * ((p.bh * runs * tiles + 7) / 8));
}

}  // namespace
