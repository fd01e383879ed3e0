// Arguments and launcher of the decode-shaped (at most 128 rows) GEMM, see skinny_kernels.hip.
#pragma once
#include "common.h"
#include "gemm.h"
#include "lora.h"

namespace mmd8 {

constexpr int kSkinnyMaxM = 128;

struct SkinnyPlan {
  int n_slabs, tiles_n, splits, slabs_per_split;
};
// how the K range is split between workgroups for this shape (depends on the device's CU count)
SkinnyPlan plan_skinny(int K, int N);

struct SkinnyArgs {
  const int8_t* Xq;       // activation codes, blocked layout, panel 0; codes of critical columns may hold anything
  const int8_t* Wt;       // weight codes, blocked layout
  const uint8_t* mask;    // [Kpad] column flags, 1 = critical column
  int M, N, Kpad;
  const float* r;         // [M]
  const float* c;         // [N]
  const uint16_t* bias;   // [N] or null
  uint16_t* Y;
  int ldy;
  float* partial;         // fp32 [splits][M][N]
  int32_t* tap_acc;       // [M][N] or null
  uint8_t* flag_reset;    // [Kpad] column flags: zeroed again by the last kernel of the call
  const float* lora_P;    // low-rank term T B^T added to the output: T as sums of lora_splits ranges (sum_low_rank_activation), B [N][lora_r] fp16
  const uint16_t* lora_B;
  int lora_splits, lora_r;   // lora_r == 0: none
  uint16_t* lora_T_user;  // [M][lora_r] or null: receives T
  // The output with a residual added, H = f16(Y + residual), and / or leaving in blockwise-coded form (the rows
  // of this call as one flattened tensor of M N elements; Y, where given, is then contiguous: ldy == N).
  const uint16_t* residual;   // [M][ldr] fp16 or null
  int ldr;
  int gelu;               // 1: Y := f16(gelu(Y)) before a residual is added
  uint8_t* codes;         // [M N] or null
  float* code_absmax;     // [ceil(M N / code_block)]
  int code_block;         // a multiple of 64, at most 4096
  const uint16_t* X;      // [M][ldx] fp16
  int ldx, K;
  uint32_t th;            // fp16 pattern of the threshold (k_gemm_rows)
  int n_slabs, tiles_n, slabs_per_split;   // filled by the launcher
};
hipError_t launch_gemm_skinny(SkinnyArgs a, const SkinnyPlan& plan, hipStream_t stream);
// Up to eight rows, the kernel that prepares its own operands and splits K (k_gemm_panel); splits 0: not for this call.
constexpr int kPanelMaxM = 8;
SkinnyPlan plan_panel(int M, int K, int N);
hipError_t launch_gemm_panel(SkinnyArgs a, const SkinnyPlan& plan, hipStream_t stream);

// Y = f16(sum of the ranges of K, in order, + bias), then GELU, then the residual; with codes, the result (also stored
// in Y, contiguous, where given) leaves blockwise-coded.
struct SplitSum {
  const float* partial;       // [splits][M][N]
  int splits, M, N;           // N a multiple of 8
  const uint16_t* bias;
  const uint16_t* residual;   // [M][ldr] or null
  int ldr;
  int gelu;
  uint16_t* Y;
  int ldy;
  uint8_t* codes;             // or null
  float* code_absmax;
  int code_block;
};
hipError_t launch_add_splits(const SplitSum& s, hipStream_t stream);

// A few rows, whole layer in one kernel (k_gemm_rows): nothing is split between workgroups and no second kernel adds
// partial outputs.  The rows' codes and fp16 critical columns for the whole of K live in LDS (3 bytes per element, as
// many rows as fit).  Needs a.X (the kernel prepares its operands); takes bias, the low-rank term of an adapter, GELU and
// a residual; no coded output (the encoder follows it).
constexpr int kRowsMaxM = 8;
constexpr int kRowsWaves = 16;
constexpr int kRowsMaxLds = 156 * 1024;   // (of 160 KB: the kernel's fixed arrays are the rest)
bool rows_kernel_fits(int M, int Kpad, int N);
hipError_t launch_gemm_rows(SkinnyArgs a, hipStream_t stream);
hipError_t prepare_rows_kernels();     // its LDS attribute on the current device (else set by the first launch)
hipError_t prepare_skinny_kernels();   // ... and that of the other kernels for at most 128 rows

}  // namespace mmd8
