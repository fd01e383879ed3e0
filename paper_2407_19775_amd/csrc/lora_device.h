// Device side of the adapter's down-projection, shared by the kernel of its own (lora_kernels.hip) and the one that also
// clears and gathers the critical columns (activation_kernels.hip).
#pragma once
#include "lora.h"
#include "operand_layout.h"

namespace mmd8 {

constexpr int kLoraRows = 16;          // rows of X per workgroup

// Workgroups [0, t_blocks * splits): 16 rows of T each, over one of `splits` ranges of K.  Wave w takes
// the 64-column steps w, w + kWaves, ... of the range;
// in a step lane l holds, for row (or rank index) l % 16, the 16 columns 16 (l / 16) .. + 16 as two
// MFMA operands of 8 (which 8 columns meet in one MFMA does not matter: both operands use the same
// assignment).  A^T is the first operand, X^T the second, so a lane ends up with four consecutive
// rank indices of one row.  The waves' partial sums meet in LDS and are added in wave order; with P
// null (one range) the sum is rounded and stored, else it goes to P[range][m][64] as fp32, and a later kernel adds the ranges in
// index order (so the result does not depend on timing) and rounds: the one that clears the critical columns or k_lora_reduce
// (reduce_low_rank_activation), for at most 128 rows the one that adds the low-rank term (sum_low_rank_activation).
// Workgroups from t_blocks * splits on copy B into the weight-side slabs.
// eight sums of row m (rank indices 8 ch .. + 8; exact zeros past the rank): rounded to fp16 and stored as
// part of T, of the caller's copy of T and of the activation-side slabs
__device__ inline void store_low_rank_activation(const LoraArgs& a, int m, int ch, const float (&sum)[8]) {
  uint32_t out[4] = {0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < 8; ++e) out[e >> 1] |= float_to_half_bits(sum[e]) << (16 * (e & 1));
  const v4u v = {out[0], out[1], out[2], out[3]};
  const int j0 = 8 * ch;
  *reinterpret_cast<v4u*>(a.T + (size_t)m * kLoraMaxRank + j0) = v;
  if (a.T_user && j0 < a.r) *reinterpret_cast<v4u*>(a.T_user + (size_t)m * a.r + j0) = v;
  if (a.Xo)
    *reinterpret_cast<v4u*>(reinterpret_cast<int8_t*>(a.Xo) + packed_chunk_offset(m, a.crit_slabs + ch / 4, ch % 4, a.f_slabs)) = v;
}

// Item (row, 8 rank indices) of T: the ranges' sums in index order, then as with one range.
__device__ inline void reduce_low_rank_activation(const LoraArgs& a, int item, int splits, const float* __restrict__ P) {
  const int n_chunks = 4 * lora_slabs(a.r);
  if (item >= a.M * n_chunks) return;
  const int m = item / n_chunks, ch = item % n_chunks;
  float sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int s = 0; s < splits; ++s) {
    const float* p = P + ((size_t)s * a.M + m) * kLoraMaxRank + 8 * ch;
    const v4f lo = *reinterpret_cast<const v4f*>(p), hi = *reinterpret_cast<const v4f*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sum[e] += lo[e];
      sum[4 + e] += hi[e];
    }
  }
  store_low_rank_activation(a, m, ch, sum);
}

// What lane group kq reads in 64-column step s of a range that ends at step `end`: 16 columns, lora_lane_column + lora_step_column
// on.  A group beyond the range or the end of the row (lora_reads false) masks what it reads, and that is within the row too.
__host__ __device__ __forceinline__ bool lora_reads(int s, int end, int kq, int K) { return s < end && 64 * s + 16 * kq < K; }
__host__ __device__ __forceinline__ int lora_lane_column(int kq, int K) { return 16 * kq < K ? 16 * kq : K - 16; }
__host__ __device__ __forceinline__ int lora_step_column(int s, bool reads) { return reads ? 64 * s : 0; }

// kTiles: 16-wide tiles of the rank, ceil(r / 16); kU: steps whose loads a wave has in flight together.  Called by every
// thread of a workgroup of kWaves waves.
template <int kTiles, int kWaves, int kU>
__device__ __forceinline__ void lora_down_block(const LoraArgs& a, int block, int t_blocks, int splits, int steps_per_split, float* __restrict__ P) {
  constexpr int kCols = kTiles * 16, kThreadsOfBlock = kWaves * kWave;
  __shared__ __attribute__((aligned(16))) float s_part[kWaves][kLoraRows][kCols];
  static_assert(kThreadsOfBlock >= kLoraRows * kLoraMaxRank / 8, "a thread per eight sums");
  const int n_chunks = 4 * lora_slabs(a.r);                         // 8-column chunks of the slabs
  if (block >= t_blocks * splits) {
    const int item = (block - t_blocks * splits) * kThreadsOfBlock + (int)threadIdx.x;
    if (a.Wo == nullptr || item >= a.N * n_chunks) return;
    const int ch = item / a.N, n = item % a.N;
    v4u v = {0, 0, 0, 0};
    if (8 * ch < a.r) v = *reinterpret_cast<const v4u*>(a.B + (size_t)n * a.r + 8 * ch);
    *reinterpret_cast<v4u*>(reinterpret_cast<int8_t*>(a.Wo) + packed_chunk_offset(n, a.crit_slabs + ch / 4, ch % 4, a.f_slabs)) = v;
    return;
  }
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
  const int m0 = (block % t_blocks) * kLoraRows, split = block / t_blocks;
  const int li = lane & 15, kq = lane >> 4;
  const int lane_column = lora_lane_column(kq, a.K);
  const uint16_t* xrow = a.X + (size_t)min(m0 + li, a.M - 1) * a.ldx + lane_column;
  const uint16_t* arow[kTiles];
  bool jvalid[kTiles];
#pragma unroll
  for (int t = 0; t < kTiles; ++t) {
    const int j = 16 * t + li;
    jvalid[t] = j < a.r;
    arow[t] = a.A + (size_t)min(j, a.r - 1) * a.K + lane_column;
  }
  v4f acc[kTiles];
#pragma unroll
  for (int t = 0; t < kTiles; ++t) acc[t] = v4f{0, 0, 0, 0};

  const int steps = min(ceil_div(a.K, 64), (split + 1) * steps_per_split);   // end of this range
  for (int s0 = split * steps_per_split + wave; s0 < steps; s0 += kWaves * kU) {
    v4u xf[kU][2], af[kU][kTiles][2];
    // every load is issued before the first use; a step past the end re-reads step 0 and is masked
#pragma unroll
    for (int u = 0; u < kU; ++u) {
      const int s = s0 + u * kWaves;
      const bool ok = lora_reads(s, steps, kq, a.K);
      const int k = lora_step_column(s, ok);
      const uint32_t keep = ok ? 0xffffffffu : 0u;
#pragma unroll
      for (int h = 0; h < 2; ++h) xf[u][h] = *reinterpret_cast<const v4u*>(xrow + k + 8 * h) & keep;
#pragma unroll
      for (int t = 0; t < kTiles; ++t) {
        const uint32_t keep_a = (ok && jvalid[t]) ? 0xffffffffu : 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h) af[u][t][h] = *reinterpret_cast<const v4u*>(arow[t] + k + 8 * h) & keep_a;
      }
    }
#pragma unroll
    for (int u = 0; u < kU; ++u)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int t = 0; t < kTiles; ++t)
          acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, af[u][t][h]),
                                                          __builtin_bit_cast(v8h, xf[u][h]), acc[t], 0, 0, 0);
  }
  // lane: row li, rank indices 16 t + 4 kq .. + 4
#pragma unroll
  for (int t = 0; t < kTiles; ++t) *reinterpret_cast<v4f*>(&s_part[wave][li][16 * t + 4 * kq]) = acc[t];
  __syncthreads();

  const int item = threadIdx.x;
  if (item >= kLoraRows * n_chunks) return;
  const int m = m0 + item / n_chunks, ch = item % n_chunks, j0 = 8 * ch;
  if (m >= a.M) return;
  float sum[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (j0 < kCols) {
    for (int w = 0; w < kWaves; ++w) {
      const v4f lo = *reinterpret_cast<const v4f*>(&s_part[w][item / n_chunks][j0]);
      const v4f hi = *reinterpret_cast<const v4f*>(&s_part[w][item / n_chunks][j0 + 4]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sum[e] += lo[e];
        sum[4 + e] += hi[e];
      }
    }
  }
  if (P) {
    float* p = P + ((size_t)split * a.M + m) * kLoraMaxRank + j0;
    *reinterpret_cast<v4f*>(p) = v4f{sum[0], sum[1], sum[2], sum[3]};
    *reinterpret_cast<v4f*>(p + 4) = v4f{sum[4], sum[5], sum[6], sum[7]};
    return;
  }
  store_low_rank_activation(a, m, ch, sum);
}

}  // namespace mmd8
