// Low-rank adapter W' = W + B A on top of the int8 layer ("BSNS with parameter-efficient
// fine-tuning via adapters"): Y = (int8 layer)(X) + T B^T with T = f16(X A^T).
//
// k_lora_down computes T on the matrix cores (v_mfma_f32_16x16x32_f16, fp32 accumulation, one
// rounding to fp16) and lays T and B out as extra fp16 slabs behind the slabs of the critical columns,
// so that the GEMM kernel adds T B^T exactly as it adds the critical columns: more fp16 MFMAs onto
// the dequantized accumulators.  For decode shapes T is kept as a plain matrix and the product
// with B is added by the kernel that sums the split-K partial outputs.
#include "lora_device.h"

namespace mmd8 {

namespace {
constexpr int kLoraThreads = 512;

template <int kTiles>
__global__ __launch_bounds__(kLoraThreads) void k_lora_down(const LoraArgs a, int t_blocks, int splits, int steps_per_split,
                                                            float* __restrict__ P) {
  lora_down_block<kTiles, kLoraThreads / kWave, (kTiles <= 2 ? 4 : 2)>(a, blockIdx.x, t_blocks, splits, steps_per_split, P);
}

// one thread per (row, 8 rank indices)
__global__ __launch_bounds__(256) void k_lora_reduce(const LoraArgs a, int splits, const float* __restrict__ P) {
  reduce_low_rank_activation(a, blockIdx.x * 256 + threadIdx.x, splits, P);
}
}  // namespace

// the host's view of the down-projection's reads: first of the 16 columns
int lora_read_column(int s, int end, int kq, int K) { return lora_lane_column(kq, K) + lora_step_column(s, lora_reads(s, end, kq, K)); }

LoraPlan plan_lora(int M, int K, bool split) {
  // K is split until there are two workgroups per compute unit, every range at least sixteen 64-column steps: the sums are
  // added in a launch that runs anyway.
  const int t_blocks = ceil_div(M, kLoraRows), steps = ceil_div(K, 64), cus = device_cu_count();
  // Up to 128 rows are a few tiles, and 16 rows and A through one compute unit take 4.5 us at K = 4096: there the ranges
  // are short (four steps) and their sums are added by the kernel that needs them, without a launch in between (7B-shaped layer with rank 16:
  // one row 74 -> 61.5 us, 32 rows 128 -> 112, 128 rows 198 -> 184; rank 64 at 64 rows 265 -> 179).
  LoraPlan p;
  p.decode = M <= 128;
  const int want = p.decode ? max(1, min(steps / 4, kLoraDecodeSplits)) : split ? max(1, min(min(2 * cus / t_blocks, steps / 16), 32)) : 1;
  p.steps_per_split = ceil_div(steps, want);
  p.splits = ceil_div(steps, p.steps_per_split);
  p.partial_bytes = p.splits > 1 || p.decode ? (size_t)p.splits * M * kLoraMaxRank * sizeof(float) : 0;
  return p;
}

hipError_t launch_lora_down(const LoraArgs& a, const LoraPlan& plan, float* partial, hipStream_t stream) {
  const int t_blocks = ceil_div(a.M, kLoraRows);
  const int b_blocks = a.Wo ? ceil_div(a.N * 4 * lora_slabs(a.r), kLoraThreads) : 0;
  if (plan.decode && !partial) return hipErrorInvalidValue;
  const dim3 grid(t_blocks * plan.splits + b_blocks), block(kLoraThreads);
  switch (ceil_div(a.r, 16)) {
    case 1: hipLaunchKernelGGL(k_lora_down<1>, grid, block, 0, stream, a, t_blocks, plan.splits, plan.steps_per_split, plan.splits > 1 || plan.decode ? partial : nullptr); break;
    case 2: hipLaunchKernelGGL(k_lora_down<2>, grid, block, 0, stream, a, t_blocks, plan.splits, plan.steps_per_split, plan.splits > 1 || plan.decode ? partial : nullptr); break;
    case 3: hipLaunchKernelGGL(k_lora_down<3>, grid, block, 0, stream, a, t_blocks, plan.splits, plan.steps_per_split, plan.splits > 1 || plan.decode ? partial : nullptr); break;
    case 4: hipLaunchKernelGGL(k_lora_down<4>, grid, block, 0, stream, a, t_blocks, plan.splits, plan.steps_per_split, plan.splits > 1 || plan.decode ? partial : nullptr); break;
    default: return hipErrorInvalidValue;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || plan.splits == 1 || plan.decode) return e;
  hipLaunchKernelGGL(k_lora_reduce, dim3(ceil_div(a.M * 4 * lora_slabs(a.r), 256)), dim3(256), 0, stream, a, plan.splits, partial);
  return hipGetLastError();
}

}  // namespace mmd8
