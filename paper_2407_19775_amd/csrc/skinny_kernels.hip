// Decode-shaped (at most 64 tokens) mixed int8 GEMM ("Compression techniques", item 2): bound by
// streaming the int8 weights once from HBM, not by the matrix pipes.
//
//   acc[m,n] = sum_k Xq[m,k] Wt[n,k]                                   v_mfma_i32_32x32x32_i8
//   Y[m,n]   = f16( acc r[m] c[n] / 127^2 + sum_{k critical} X[m,k] f16(Wt[n,k] c[n]/127) + bias[n] )
//
// No weight byte is used by more than one wave, so the weights go straight from HBM into the
// registers of the lane that feeds them to the MFMA (no LDS): a wave owns 32 rows of Wt (32 output
// columns) and reads their 64-byte slabs; the blocked layout is fragment-major, so each of the two
// loads per slab is 1 KB of consecutive addresses.  The activation side of a slab is shared by the
// waves of a workgroup through LDS.  When there are too few weight panels to give every CU a
// workgroup, the K range is split between workgroups, which write fp32 partial outputs that a
// second small kernel adds in a fixed order (the result does not depend on timing).
//
// Heavy-tailed decode activations flag a large share of the feature dimensions, so the 16-bit part
// is a second product over the same weights rather than a small correction.  For a slab that holds
// a critical column the lane turns the weight bytes it already has into fp16 and multiplies them
// with Xf, a copy of X in which the non-critical columns are zero (written by the pack kernel).
// To keep that conversion off the critical path the fp16 operand is the integer code itself (exact
// in fp16, one byte permute and one packed fp16 subtraction per two codes) and the column step
// c[n]/127 is applied in fp32 to the accumulated sum: the sum over the critical columns of
// X[m,k] q[n,k] c[n]/127 with one rounding at the end, instead of rounding each dequantized weight
// to fp16 first.  The two differ by at most the fp16 rounding of the weights (2^-11 relative per
// term), far inside the tolerance of the fp16 output.  A slab without a critical column skips the
// 16-bit part (the same decision for the whole workgroup).
#include <type_traits>
#include <utility>

#include <atomic>

#include "codec_device.h"
#include "common.h"
#include "operand_layout.h"
#include "skinny.h"

namespace mmd8 {

// ------------------------------------------------------------------------------------------------
// If every wave fetched its own copy of the activation fragments from L2, that would be up to 6
// times the bytes of the weights it streams (64 rows).  So the kWaves waves of a workgroup own
// neighbouring 32-column groups of one weight panel and walk the same slabs together: the
// activation side of a slab (int8 codes and the fp16 critical columns, kMT 32-row groups each) is
// fetched once per workgroup, parked in LDS (a ring of four buffers) and read from there by every
// wave; the weights go from HBM straight into the registers of the lane that feeds them to the
// MFMA, three slabs ahead.  All waits are the compiler's.  Measured per workgroup: about 19 GB/s
// of weights at 64 rows (the MFMAs and the code-to-fp16 conversions of a slab take about as long
// as its 16 KB take to arrive), so every CU must have a workgroup.
// ------------------------------------------------------------------------------------------------
template <int MT, int WAVES>
struct PanelCfg {
  static constexpr int kMT = MT, kWaves = WAVES;
  static constexpr int kThreads = WAVES * kWave;
  static constexpr int kCols = WAVES * 32;
  static constexpr int XQ_BYTES = MT * 2048, XF_BYTES = MT * 4096, STAGE_BYTES = XQ_BYTES + XF_BYTES;
  static constexpr int kPieces = STAGE_BYTES / 1024;               // 1 KB pieces of a slab's activation side
  static constexpr int kFetch = (kPieces + WAVES - 1) / WAVES;     // per wave and slab; surplus ones repeat the last
  static constexpr int kMaxSlabs = MMD8_MAX_K / kSlabBytes;        // flags "slab holds a critical column"
};

// kPrep (at most kPanelPrepMaxM rows): the activation side is not fetched from packed operands but made here.
// Every workgroup streams the rows of X once for the row scales (the maximum of the magnitudes below the
// threshold, as the scan kernel finds it), keeps the columns of its own K range in LDS with one "critical" flag
// per column, and writes the codes and the fp16 critical columns of a slab into the ring two slabs ahead of the
// MFMAs: wave w owns the 16-column piece w % 4 of the slab, a lane one column of one of four rows.  The
// arithmetic is the pack kernel's (IEEE 127 / r, rint, clamp; critical columns zero in the codes and kept in the
// fp16 copy).  Rows of the ring beyond M are zeroed once and never written.
template <class Cfg, bool kSplit, bool kTap, bool kPrep>
__global__ __launch_bounds__(Cfg::kThreads, 2) void k_gemm_panel(const SkinnyArgs a) {
  constexpr int MT = Cfg::kMT, WAVES = Cfg::kWaves;
  static_assert(!kPrep || MT == 1, "own preparation is for a few rows");
  __shared__ __attribute__((aligned(16))) int8_t s_x[4][Cfg::STAGE_BYTES];
  __shared__ uint8_t s_any[Cfg::kMaxSlabs];
  __shared__ __attribute__((aligned(16))) uint16_t s_row[kPrep ? kPanelPrepMaxRowSlabs * kSlabBytes : 8];   // [M][cnt x 64]
  __shared__ __attribute__((aligned(16))) uint8_t s_crit[kPrep ? kPanelPrepMaxSlabs * kSlabBytes : 16];                                    // [cnt x 64]
  __shared__ uint32_t s_part[kPanelPrepMaxM][WAVES];
  __shared__ float s_r[kPanelPrepMaxM], s_scale[kPanelPrepMaxM];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lr = lane & 31, lg = lane >> 5;
  reset_column_flags(a.flag_reset, a.Kpad);
  const int tile = blockIdx.x % a.tiles_n, split = blockIdx.x / a.tiles_n;
  const int n0 = tile * Cfg::kCols + wave * 32;                    // < Npad: the padding rows of Wt are zero
  const int n = n0 + lr;
  const int s_begin = split * a.slabs_per_split;
  const int cnt = min(a.n_slabs, s_begin + a.slabs_per_split) - s_begin;   // >= 1 by construction of the plan

  const int8_t* wgrp = a.Wt + (size_t)(n0 >> 8) * a.n_slabs * kBlockBytes + (size_t)((n0 & 255) >> 5) * 2048 + lane * 16 +
                       (size_t)s_begin * kBlockBytes;
  if constexpr (!kPrep) {
    for (int t = threadIdx.x; t < cnt; t += Cfg::kThreads) {
      const v4u* mk = reinterpret_cast<const v4u*>(a.mask + (size_t)(s_begin + t) * kSlabBytes);
      const v4u m = mk[0] | mk[1] | mk[2] | mk[3];
      s_any[t] = (m[0] | m[1] | m[2] | m[3]) != 0;
    }
  }

  // piece i of a slab's activation side: first the int8 codes (MT 32-row groups x 2 k-steps), then
  // the fp16 pieces (MT groups x 4); the first MT groups of a slab are contiguous in both arrays
  const int8_t* x_src[Cfg::kFetch];
  int x_dst[Cfg::kFetch], x_step[Cfg::kFetch];
#pragma unroll
  for (int d = 0; d < Cfg::kFetch; ++d) {
    const int i = min(wave + d * WAVES, Cfg::kPieces - 1);
    const bool codes = i < MT * 2;
    x_src[d] = (codes ? a.Xq + (size_t)s_begin * kBlockBytes + i * 1024
                      : reinterpret_cast<const int8_t*>(a.Xf) + (size_t)s_begin * 8192 + (i - MT * 2) * 1024) + lane * 16;
    x_step[d] = codes ? kBlockBytes : 8192;
    x_dst[d] = i * 1024 + lane * 16;
  }
  auto fetch_x = [&](int j, v4i (&xr)[Cfg::kFetch]) {
    if constexpr (kPrep) return;
#pragma unroll
    for (int d = 0; d < Cfg::kFetch; ++d) xr[d] = *reinterpret_cast<const v4i*>(x_src[d] + (size_t)j * x_step[d]);
  };
  // kPrep: slab j of the workgroup's range -> ring buffer `stage` (see the kernel's header comment)
  const int row_stride = cnt * kSlabBytes;                         // elements of s_row per row
  auto make_slab = [&](int j, int stage) {
    const int ch = wave & 3, ks = ch >> 1, g = ch & 1, col = lane & 15;
    const int kl = j * kSlabBytes + ch * 16 + col;
    const bool crit = s_crit[kl] != 0;
    for (int m = (wave >> 2) * 4 + (lane >> 4); m < a.M; m += WAVES) {
      const uint32_t x = s_row[m * row_stride + kl];
      const uint32_t code = crit ? 0u : to_code_byte(half_lo_to_float(x), s_scale[m]);
      s_x[stage][ks * 1024 + (32 * g + m) * 16 + col] = (int8_t)code;
      *reinterpret_cast<uint16_t*>(&s_x[stage][Cfg::XQ_BYTES + (2 * ks + (col >> 3)) * 1024 + (32 * g + m) * 16 +
                                               (col & 7) * 2]) = crit ? (uint16_t)x : (uint16_t)0;
    }
  };
  auto park_x = [&](int stage, const v4i (&xr)[Cfg::kFetch], int j) {   // j: the slab these pieces belong to
    if constexpr (kPrep) {
      make_slab(j, stage);
    } else {
#pragma unroll
      for (int d = 0; d < Cfg::kFetch; ++d) *reinterpret_cast<v4i*>(&s_x[stage][x_dst[d]]) = xr[d];
    }
  };
  struct W2 {
    v4i w[2];
  };
  auto fetch_w = [&](int j, W2& f) {
    const int8_t* p = wgrp + (size_t)j * kBlockBytes;
    f.w[0] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
    f.w[1] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p + 1024));
  };

  v16i acc[MT];
  v16f accf[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[mt][e] = 0, accf[mt][e] = 0.0f;

  struct Frags {
    v4i x[MT][2];      // int8 codes, k-steps 0 and 1
    v8h xf[MT][4];     // fp16 critical columns, pieces 2 ks + t (valid when the slab has any)
  };
  auto read_frags = [&](int stage, bool any, Frags& g) {
    const int8_t* base = &s_x[stage][lane * 16];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) g.x[mt][ks] = *reinterpret_cast<const v4i*>(base + mt * 2048 + ks * 1024);
    if (any) {                                                     // the same for the whole workgroup
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int p = 0; p < 4; ++p)
          g.xf[mt][p] = *reinterpret_cast<const v8h*>(base + Cfg::XQ_BYTES + mt * 4096 + p * 1024);
    }
  };
  auto multiply = [&](bool any, const Frags& g, const W2& f) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = __builtin_amdgcn_mfma_i32_32x32x32_i8(g.x[mt][ks], f.w[ks], acc[mt], 0, 0, 0);
    if (any) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const v4u wu = __builtin_bit_cast(v4u, f.w[ks]) ^ 0x80808080u;
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const v8h wh = codes_to_half8(wu, t);
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) accf[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(g.xf[mt][2 * ks + t], wh, accf[mt], 0, 0, 0);
        }
      }
    }
  };

  // Software pipeline (past the end the requests repeat the last slab: L2 hits, uniform loop body).
  // In iteration j: request the activation pieces of slab j + 5 and the weights of slab j + 3; read the fragments
  // of slab j + 1 from LDS (they overlap the MFMAs of slab j, whose fragments were read an iteration
  // ago); park the pieces of slab j + 2 (requested three iterations ago) in the buffer that slab j - 1
  // used (a ring of four, so that every index is static in a loop unrolled four times); barrier.
  const int last = cnt - 1;
  W2 f[4];
  // Activation pieces on their way from L2 to LDS: slab s >= 1 travels in xr[s % 4] (slab 0 in x0), requested three
  // iterations before it is parked (the pieces were written by another kernel, possibly through another XCD's
  // L2; four registers per set).
  v4i x0[Cfg::kFetch], xr[4][Cfg::kFetch];
  Frags fr[2];
  // (requests in the order the loop issues them, so that what the compiler counts as in flight on entry to the
  // loop is what it counts when coming round)
  fetch_x(0, x0);
  fetch_x(min(1, last), xr[1]);
  fetch_x(min(2, last), xr[2]);
  fetch_w(0, f[0]);
  fetch_x(min(3, last), xr[3]);
  fetch_w(min(1, last), f[1]);
  fetch_x(min(4, last), xr[0]);
  fetch_w(min(2, last), f[2]);
  if constexpr (kPrep) {
    // (the weight requests above are in flight meanwhile)
    for (int i = threadIdx.x; i < 4 * Cfg::STAGE_BYTES / 16; i += Cfg::kThreads)
      reinterpret_cast<v4u*>(&s_x[0][0])[i] = v4u{0, 0, 0, 0};
    const us2 th2 = __builtin_bit_cast(us2, a.th | (a.th << 16));
    // rows innermost, so that the loads of all rows are in flight together
    us2 best[kPanelPrepMaxM];
#pragma unroll
    for (int m = 0; m < kPanelPrepMaxM; ++m) best[m] = __builtin_bit_cast(us2, 0u);
    for (int c = threadIdx.x; c < a.K / 8; c += Cfg::kThreads) {
      v4u raw[kPanelPrepMaxM];
#pragma unroll
      for (int m = 0; m < kPanelPrepMaxM; ++m) {
        raw[m] = v4u{0, 0, 0, 0};
        if (m < a.M) raw[m] = *reinterpret_cast<const v4u*>(a.X + (size_t)m * a.ldx + c * 8);
      }
#pragma unroll
      for (int m = 0; m < kPanelPrepMaxM; ++m)
#pragma unroll
        for (int w = 0; w < 4; ++w)   // per half, wraps mod 2^16: entries below the threshold get the top bit
          best[m] = __builtin_elementwise_max(best[m], (us2)(__builtin_bit_cast(us2, raw[m][w] & 0x7fff7fffu) - th2));
    }
    // this workgroup's columns (the K padding reads as zero)
    for (int c = threadIdx.x; c < cnt * (kSlabBytes / 8); c += Cfg::kThreads) {
      const int k = s_begin * kSlabBytes + c * 8;
      v4u raw[kPanelPrepMaxM];
#pragma unroll
      for (int m = 0; m < kPanelPrepMaxM; ++m) {
        raw[m] = v4u{0, 0, 0, 0};
        if (m < a.M && k < a.K) raw[m] = *reinterpret_cast<const v4u*>(a.X + (size_t)m * a.ldx + k);
      }
#pragma unroll
      for (int m = 0; m < kPanelPrepMaxM; ++m)
        if (m < a.M) *reinterpret_cast<v4u*>(&s_row[m * row_stride + c * 8]) = raw[m];
    }
#pragma unroll
    for (int m = 0; m < kPanelPrepMaxM; ++m) {
      if (m < a.M) {                                                  // the same for every lane
        const uint32_t both = __builtin_bit_cast(uint32_t, best[m]);
        const uint32_t wmax = wave_max_u32(max(both & 0xffffu, both >> 16));
        if (lane == 0) s_part[m][wave] = wmax;
      }
    }
    __syncthreads();
    for (int c = threadIdx.x; c < row_stride; c += Cfg::kThreads) {
      bool crit = false;
      for (int m = 0; m < a.M; ++m) crit = crit || (s_row[m * row_stride + c] & 0x7fffu) >= a.th;
      s_crit[c] = crit ? 1 : 0;
    }
    if ((int)threadIdx.x < a.M) {
      uint32_t mm = 0;
#pragma unroll
      for (int w = 0; w < WAVES; ++w) mm = max(mm, s_part[threadIdx.x][w]);
      // top bit set: an entry below the threshold exists and its pattern is mm + th (mod 2^16)
      const float r = (mm & 0x8000u) ? half_lo_to_float((mm + a.th) & 0xffffu) : 0.0f;
      s_r[threadIdx.x] = r;
      s_scale[threadIdx.x] = (r == 0.0f) ? 0.0f : 127.0f / r;       // IEEE division
    }
    __syncthreads();
    for (int t = threadIdx.x; t < cnt; t += Cfg::kThreads) {         // "slab t holds a critical column"
      const v4u* fl = reinterpret_cast<const v4u*>(&s_crit[t * kSlabBytes]);
      const v4u m = fl[0] | fl[1] | fl[2] | fl[3];
      s_any[t] = (m[0] | m[1] | m[2] | m[3]) != 0;
    }
  }
  park_x(0, x0, 0);
  park_x(1, xr[1], min(1, last));
  __syncthreads();
  // The flags of the next 64 slabs as one scalar mask (bit i: slab base + i, the last slab repeated past the end),
  // refilled every 64 iterations: no LDS read and no vector compare between a slab's fragments and its MFMAs.
  uint64_t any_mask = __builtin_amdgcn_ballot_w64(s_any[min(lane, last)] != 0);
  bool any_next = any_mask & 1u;
  read_frags(0, any_next, fr[0]);
  auto iteration = [&](int j, auto u_tag) {
    constexpr int u = decltype(u_tag)::value;                        // j % 4
    const bool any_cur = any_next;
    if constexpr (u == 3) {                                          // 64 is a multiple of four: only here can j + 1 start a window
      if (((j + 1) & 63) == 0) any_mask = __builtin_amdgcn_ballot_w64(s_any[min(j + 1 + lane, last)] != 0);
    }
    any_next = (any_mask >> ((j + 1) & 63)) & 1u;
    fetch_x(min(j + 5, last), xr[(u + 1) & 3]);
    fetch_w(min(j + 3, last), f[(u + 3) & 3]);
    read_frags((u + 1) & 3, any_next, fr[(u + 1) & 1]);
    multiply(any_cur, fr[u & 1], f[u & 3]);
    park_x((u + 2) & 3, xr[(u + 2) & 3], min(j + 2, last));
    __syncthreads();
  };
  // Whole groups of four iterations run without a way out in between: with an exit after every iteration the
  // compiler's count of the requests still in flight is merged over all those paths, and it then waits for
  // weights requested one iteration earlier instead of three (every iteration took a whole memory latency).
  int j0 = 0;
  for (; j0 + 4 <= cnt; j0 += 4) {
    iteration(j0, std::integral_constant<int, 0>{});
    iteration(j0 + 1, std::integral_constant<int, 1>{});
    iteration(j0 + 2, std::integral_constant<int, 2>{});
    iteration(j0 + 3, std::integral_constant<int, 3>{});
  }
  if (j0 < cnt) iteration(j0, std::integral_constant<int, 0>{});
  if (j0 + 1 < cnt) iteration(j0 + 1, std::integral_constant<int, 1>{});
  if (j0 + 2 < cnt) iteration(j0 + 2, std::integral_constant<int, 2>{});

  // ---- outputs.  C layout of the 32x32 MFMA: lane = column n (lane % 32), register e = row
  // 8 (e / 4) + 4 (lane / 32) + (e % 4).
  const float cs = (n < a.N) ? a.c[n] / 16129.0f : 0.0f;
  const float step = (n < a.N) ? a.c[n] / 127.0f : 0.0f;
  const float b = (!kSplit && a.bias && n < a.N) ? half_lo_to_float(a.bias[n]) : 0.0f;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int m = mt * 32 + 8 * (e >> 2) + 4 * lg + (e & 3);
      if (m < a.M && n < a.N) {
        const float rm = kPrep ? s_r[m] : a.r[m];
        const float y = (float)acc[mt][e] * (rm * cs) + accf[mt][e] * step;
        if constexpr (kSplit)
          a.partial[((size_t)split * a.M + m) * a.N + n] = y;
        else
          a.Y[(size_t)m * a.ldy + n] = (uint16_t)float_to_half_bits(y + b);
        if constexpr (kTap) {
          if constexpr (kSplit)
            atomicAdd(a.tap_acc + (size_t)m * a.N + n, acc[mt][e]);   // tap buffer zeroed by the launcher
          else
            a.tap_acc[(size_t)m * a.N + n] = acc[mt][e];
        }
      }
    }
}

// kCols neighbouring sums of `splits` ranges, added in index order, eight loads in flight at a time.  (Added one load
// after the other, sixteen ranges cost the kernel sixteen memory latencies.)
template <int kCols>
__device__ __forceinline__ void add_ranges(const float* __restrict__ p, int splits, size_t MN, float (&y)[kCols]) {
  static_assert(kCols == 1 || kCols == 4, "a dword or four");
  typedef typename std::conditional<kCols == 1, float, v4f>::type Piece;
  auto add = [&](const Piece& q) {
    if constexpr (kCols == 1) {
      y[0] += q;
    } else {
#pragma unroll
      for (int i = 0; i < kCols; ++i) y[i] += q[i];
    }
  };
#pragma unroll
  for (int i = 0; i < kCols; ++i) y[i] = 0.0f;
  int s = 0;
  auto batch = [&](auto n_tag) {
    constexpr int kN = decltype(n_tag)::value;
    Piece q[kN];
#pragma unroll
    for (int u = 0; u < kN; ++u) q[u] = *reinterpret_cast<const Piece*>(p + u * MN);
#pragma unroll
    for (int u = 0; u < kN; ++u) add(q[u]);
    s += kN;
    p += kN * MN;
  };
  while (s + 8 <= splits) batch(std::integral_constant<int, 8>{});
  if (s + 4 <= splits) batch(std::integral_constant<int, 4>{});
  if (s + 2 <= splits) batch(std::integral_constant<int, 2>{});
  if (s < splits) batch(std::integral_constant<int, 1>{});
}

// Y[m,n] = f16( sum_s partial[s][m][n] + bias[n] + sum_j T[m][j] B[n][j] ), splits added in index
// order, then the bias, then the low-rank term (T: [M][ldt] fp16, B: [N][r] fp16, r a multiple of 8;
// r == 0: no such term).  A row per blockIdx.y.
__global__ __launch_bounds__(256) void k_skinny_finalize(const float* __restrict__ partial, int splits, int M, int N,
                                                         const uint16_t* __restrict__ bias,
                                                         const uint16_t* __restrict__ T, int ldt,
                                                         const uint16_t* __restrict__ B, int r,
                                                         const uint16_t* residual /* may alias Y */, int ldr, int gelu,
                                                         uint16_t* Y, int ldy, uint8_t* flag_reset, int Kpad) {
  if (blockIdx.y == 0) reset_column_flags(flag_reset, Kpad);
  const int m = blockIdx.y, n = (int)blockIdx.x * 256 + (int)threadIdx.x;
  if (n >= N) return;
  float sum[1];
  add_ranges<1>(partial + (size_t)m * N + n, splits, (size_t)M * N, sum);
  float y = sum[0];
  if (bias) y += half_lo_to_float(bias[n]);
  if (r > 0) {
    float low = 0.0f;
    for (int j = 0; j < r; j += 8) {
      const v4u t = *reinterpret_cast<const v4u*>(T + (size_t)m * ldt + j);
      const v4u b = *reinterpret_cast<const v4u*>(B + (size_t)n * r + j);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        low += half_lo_to_float(t[e]) * half_lo_to_float(b[e]) + half_hi_to_float(t[e]) * half_hi_to_float(b[e]);
    }
    y += low;
  }
  uint32_t h = float_to_half_bits(y);
  if (gelu) h = gelu_to_half_bits(half_lo_to_float(h));
  if (residual) h = float_to_half_bits(half_lo_to_float(h) + half_lo_to_float(residual[(size_t)m * ldr + n]));
  Y[(size_t)m * ldy + n] = (uint16_t)h;
}

// The same sum as the source of the blockwise encoder (output leaving in coded form, no low-rank term): eight
// neighbouring columns of a row per call; H = f16(Y + residual) is stored where wanted and handed to the encoder.
__device__ const DynamicCode kExitCode = make_dynamic_code();
struct FinalizedHalves {
  const float* partial;
  int splits, N;
  size_t MN;
  const uint16_t* bias;
  const uint16_t* residual;
  int ldr;
  uint16_t* H;            // [M N] or null
  __device__ v4u chunk(size_t e0, int /*valid: N is a multiple of 8, chunks are whole*/) const {
    const int m = (int)(e0 / N), n = (int)(e0 % N);
    float y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = 0.0f;
    // four splits' loads in flight at a time; the additions stay in split order
    int s = 0;
    for (; s + 4 <= splits; s += 4) {
      v4f p0[4], p1[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        p0[u] = *reinterpret_cast<const v4f*>(partial + (size_t)(s + u) * MN + e0);
        p1[u] = *reinterpret_cast<const v4f*>(partial + (size_t)(s + u) * MN + e0 + 4);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] += p0[u][i], y[4 + i] += p1[u][i];
    }
    for (; s < splits; ++s) {
      const v4f p0 = *reinterpret_cast<const v4f*>(partial + (size_t)s * MN + e0);
      const v4f p1 = *reinterpret_cast<const v4f*>(partial + (size_t)s * MN + e0 + 4);
#pragma unroll
      for (int i = 0; i < 4; ++i) y[i] += p0[i], y[4 + i] += p1[i];
    }
    if (bias) {
#pragma unroll
      for (int i = 0; i < 8; ++i) y[i] += half_lo_to_float(bias[n + i]);
    }
    v4u h;
#pragma unroll
    for (int w = 0; w < 4; ++w) h[w] = float_to_half_bits(y[2 * w]) | (float_to_half_bits(y[2 * w + 1]) << 16);
    if (residual) {
      const v4u res = *reinterpret_cast<const v4u*>(residual + (size_t)m * ldr + n);
#pragma unroll
      for (int w = 0; w < 4; ++w)
        h[w] = float_to_half_bits(half_lo_to_float(h[w]) + half_lo_to_float(res[w])) |
               (float_to_half_bits(half_hi_to_float(h[w]) + half_hi_to_float(res[w])) << 16);
    }
    if (H) *reinterpret_cast<v4u*>(H + e0) = h;
    return h;
  }
};
__global__ __launch_bounds__(kCodecThreads) void k_skinny_finalize_coded(const FinalizedHalves src, int block,
                                                                         uint8_t* __restrict__ codes,
                                                                         float* __restrict__ absmax,
                                                                         int blocks_per_span, size_t n_spans,
                                                                         uint8_t* flag_reset, int Kpad) {
  reset_column_flags(flag_reset, Kpad);
  encode_spans(src, src.MN, block, codes, absmax, blocks_per_span, n_spans, kExitCode);
}

// The ranges of K of a tiled GEMM added up: four neighbouring columns of a row per thread (16-byte loads), a row
// per blockIdx.y.  Bound by the bytes of the partial sums, which the GEMM has just
// written: most are still in the last-level cache.
__global__ __launch_bounds__(256) void k_add_splits(const SplitSum a) {
  const int n = ((int)blockIdx.x * 256 + (int)threadIdx.x) * 4, m = blockIdx.y;
  if (n >= a.N) return;
  float y[4];
  add_ranges<4>(a.partial + (size_t)m * a.N + n, a.splits, (size_t)a.M * a.N, y);
  uint32_t h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = float_to_half_bits(a.bias ? y[i] + half_lo_to_float(a.bias[n + i]) : y[i]);
    if (a.gelu) h[i] = gelu_to_half_bits(half_lo_to_float(h[i]));
  }
  if (a.residual) {
    const v2u res = *reinterpret_cast<const v2u*>(a.residual + (size_t)m * a.ldr + n);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      h[i] = float_to_half_bits(half_lo_to_float(h[i]) + ((i & 1) ? half_hi_to_float(res[i >> 1]) : half_lo_to_float(res[i >> 1])));
  }
  *reinterpret_cast<v2u*>(a.Y + (size_t)m * a.ldy + n) = v2u{h[0] | (h[1] << 16), h[2] | (h[3] << 16)};
}

__global__ void k_fill_i32(int32_t* __restrict__ p, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = 0;
}

// Decode plan: `waves` neighbouring 32-column groups per workgroup.
static SkinnyPlan plan_panel(int M, int K, int N, int waves) {
  SkinnyPlan p;
  p.waves = waves;
  p.n_slabs = packed_k(K) / kSlabBytes;
  p.tiles_n = packed_n(N) / (32 * waves);
  // as many workgroups as the chip holds at once (two of four waves or one of eight per CU), every
  // workgroup with at least 8 slabs, no second round
  const int slots = device_cu_count() * (waves == 4 ? 2 : 1);
  const int want = max(1, min(p.n_slabs / 8, slots / p.tiles_n));
  p.slabs_per_split = ceil_div(p.n_slabs, want);
  p.splits = ceil_div(p.n_slabs, p.slabs_per_split);
  p.partial_bytes = p.splits > 1 ? (size_t)p.splits * M * N * sizeof(float) : 0;
  return p;
}
SkinnyPlan plan_skinny(int M, int K, int N) {
  const SkinnyPlan p4 = plan_panel(M, K, N, 4), p8 = plan_panel(M, K, N, 8);
  // measured on the Llama-7B linears: eight waves per panel beat four (half the LDS fills per weight byte)
  SkinnyPlan p = p8;
  p.partial_bytes = max(p4.partial_bytes, p8.partial_bytes);     // the workspace serves either
  return p;
}

template <class Cfg, bool kSplit, bool kTap, bool kPrep>
static hipError_t launch_panel_one(const SkinnyArgs& a, int splits, hipStream_t stream) {
  hipLaunchKernelGGL((k_gemm_panel<Cfg, kSplit, kTap, kPrep>), dim3(a.tiles_n * splits), dim3(Cfg::kThreads), 0, stream, a);
  return hipGetLastError();
}
template <class Cfg, bool kPrep>
static hipError_t launch_panel_cfg(const SkinnyArgs& a, int splits, hipStream_t stream) {
  const bool split = splits > 1 || a.lora_r > 0 || a.residual || a.codes || a.gelu, tap = a.tap_acc != nullptr;
  if (split)
    return tap ? launch_panel_one<Cfg, true, true, kPrep>(a, splits, stream)
               : launch_panel_one<Cfg, true, false, kPrep>(a, splits, stream);
  return tap ? launch_panel_one<Cfg, false, true, kPrep>(a, splits, stream)
             : launch_panel_one<Cfg, false, false, kPrep>(a, splits, stream);
}
static hipError_t launch_panel(const SkinnyArgs& a, const SkinnyPlan& plan, hipStream_t stream) {
  const bool two = a.M > 32;
  if (a.X) {                                                         // the kernel prepares its own operands
    if (two || !panel_prep_fits(a.M, plan)) return hipErrorInvalidValue;
    return plan.waves == 8 ? launch_panel_cfg<PanelCfg<1, 8>, true>(a, plan.splits, stream)
                           : launch_panel_cfg<PanelCfg<1, 4>, true>(a, plan.splits, stream);
  }
  if (plan.waves == 8)
    return two ? launch_panel_cfg<PanelCfg<2, 8>, false>(a, plan.splits, stream)
               : launch_panel_cfg<PanelCfg<1, 8>, false>(a, plan.splits, stream);
  return two ? launch_panel_cfg<PanelCfg<2, 4>, false>(a, plan.splits, stream)
             : launch_panel_cfg<PanelCfg<1, 4>, false>(a, plan.splits, stream);
}

static hipError_t launch_finalize_coded(const FinalizedHalves& src, int block, uint8_t* codes, float* absmax,
                                        uint8_t* flag_reset, int Kpad, hipStream_t stream) {
  // spans of about 2048 elements (every thread of the workgroup has a chunk), whole blocks each
  const int blocks_per_span = block >= 2048 ? 1 : 2048 / block;
  const size_t span = (size_t)blocks_per_span * block, n_spans = (src.MN + span - 1) / span;
  hipLaunchKernelGGL(k_skinny_finalize_coded, dim3((unsigned)n_spans), dim3(kCodecThreads), 0, stream, src, block, codes, absmax,
                     blocks_per_span, n_spans, flag_reset, Kpad);
  return hipGetLastError();
}

hipError_t launch_add_splits(const SplitSum& a, hipStream_t stream) {
  if (a.codes) {
    const FinalizedHalves src = {a.partial, a.splits, a.N, (size_t)a.M * a.N, a.bias, a.residual, a.ldr, a.Y};
    return launch_finalize_coded(src, a.code_block, a.codes, a.code_absmax, nullptr, 0, stream);
  }
  if (a.M > 65535) return hipErrorInvalidValue;                    // (a grid dimension; splits are for a few thousand rows at most)
  hipLaunchKernelGGL(k_add_splits, dim3(ceil_div(a.N, 1024), a.M), dim3(256), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_gemm_skinny(SkinnyArgs a, const SkinnyPlan& plan, hipStream_t stream) {
  a.n_slabs = plan.n_slabs;
  a.tiles_n = plan.tiles_n;
  a.slabs_per_split = plan.slabs_per_split;
  // with a low-rank term, an activation, a residual or a coded output the result always goes through the partial
  // buffer: the kernel that sums it adds the term, applies the activation and encodes
  const bool split = plan.splits > 1 || a.lora_r > 0 || a.residual || a.codes || a.gelu, tap = a.tap_acc != nullptr;
  const size_t n = (size_t)a.M * a.N;
  if (split && tap) hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, a.tap_acc, n);
  if (a.flag_reset_late && !split) return hipErrorInvalidValue;    // no kernel after the panel kernel to clear them
  hipError_t e = launch_panel(a, plan, stream);
  if (e != hipSuccess) return e;
  if (split && a.codes) {
    const FinalizedHalves src = {a.partial, plan.splits, a.N, n, a.bias, a.residual, a.ldr, a.Y};
    e = launch_finalize_coded(src, a.code_block, a.codes, a.code_absmax, a.flag_reset_late, a.Kpad, stream);
  } else if (split) {
    hipLaunchKernelGGL(k_skinny_finalize, dim3(ceil_div(a.N, 256), a.M), dim3(256), 0, stream, a.partial, plan.splits,
                       a.M, a.N, a.bias, a.lora_T, a.lora_ldt, a.lora_B, a.lora_r, a.residual, a.ldr, a.gelu, a.Y, a.ldy,
                       a.flag_reset_late, a.Kpad);
    e = hipGetLastError();
  }
  return e;
}

// ------------------------------------------------------------------------------------------------
// A few rows: the whole layer in one kernel.  A workgroup of sixteen waves has a compute unit to itself.  It prepares
// the activation side once, for the whole of K, as plain rows in LDS (row scales from a pass over the rows, codes with
// the critical columns zero, an fp16 copy that keeps only those), then walks its share of the 16-column tiles of the
// output (half a 32-row group of Wt each): wave w multiplies slabs w, w + 16, ... of every tile, weights straight from
// memory into registers eight slabs ahead, on from one tile to the next, with no barrier: the operands are read-only by
// then.  A lane builds its MFMA fragment from the row it stands for, lanes beyond the rows feed zeros.  The sixteen
// partial results of a tile are left in LDS and added at the end: the int32 sums are exact, the fp32 sums of the 16-bit
// part are added in wave order, so the output does not depend on timing.  No split of K between workgroups, hence no
// partial outputs in memory and no second kernel.
//
// What bounds it: the weights' bytes, and the microseconds before the first and after the last of them.  A kernel that does
// nothing but read them takes 9.1 us for 4096 x 12288 (4.0 us for 4096 x 4096, 14.6 for 4096 x 22016, 8.2 for 11008 x 4096),
// weights from memory, launch included; this one 11.9, 6.5, 18.6 and 11 at one row.
// Order of the requests: a compute unit's loads come back in the order in which they were made, so the rows of X and the
// terms of the output columns are asked for before any weight; the other way round the preparation cannot begin before
// the first weights have come from memory.  For the same reason few weights are requested ahead (48 KB per compute unit):
// with 128 KB the rows, and whatever else a wave asks for, queue behind them, and a 7B layer takes 48.5 us at one row
// instead of 45.9.  And a compute unit prepares once: with two or three workgroups on it (32 columns each) the rows of
// the second queued behind the weights of the first.  A layer of one / two / four rows took 53 / 63 / 68 us when the weights
// were requested first, in workgroups of 32 columns (four rows: with K split between workgroups); 45.9 / 52.9 / 60.9 now.
// kM: rows, at most (1, 2, 4, 8).  kChunks: 8-column chunks of the rows per thread (a number the compiler knows, so that
// they are loaded all together: a load under a condition is waited for before the next one is issued).
// ------------------------------------------------------------------------------------------------
template <int kM, int kChunks>
__global__ __launch_bounds__(kRowsWaves * kWave) void k_gemm_rows(const SkinnyArgs a) {
  constexpr int WAVES = kRowsWaves, kThreads = WAVES * kWave, kAhead = 3;
  extern __shared__ __attribute__((aligned(16))) int8_t s_ops[];     // rows_lds_bytes: operands, chunk flags, sums
  __shared__ uint8_t s_any[MMD8_MAX_K / kSlabBytes];
  __shared__ uint32_t s_part[kM][WAVES];
  __shared__ float s_r[kM], s_scale[kM];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // the operand row / output column a lane stands for, and which 16-byte piece of the slab it holds
  const int lr = lane & 15, lg = lane >> 4;
  const int n_slabs = a.n_slabs, Kpad = n_slabs * kSlabBytes;
  const int M = kM == 1 ? 1 : a.M;
  reset_column_flags(a.flag_reset, Kpad);
  const int row_chunks = Kpad / 8, all_chunks = M * row_chunks;
  int8_t* s_code = s_ops;                                            // [M][Kpad]
  uint16_t* s_xf = reinterpret_cast<uint16_t*>(s_ops + (size_t)M * Kpad);    // [M][Kpad]
  uint8_t* s_over = reinterpret_cast<uint8_t*>(s_xf + (size_t)M * Kpad);     // [all_chunks]: bits "at or above the threshold" (kM > 1)
  int32_t* s_sum = reinterpret_cast<int32_t*>(s_over + (kM > 1 ? round_up(all_chunks, 16) : 0));   // [tile][int / float][wave][M][16]
  const int tile_words = 2 * WAVES * M * 16;

  // ---- the rows, read once: a thread keeps its chunks (rows and columns flattened) in registers from the pass that finds
  // the row scales to the pass that writes codes and fp16 critical columns
  v4u raw[kChunks];
  auto chunk_place = [&](int i, int& m, int& c) {                     // false: beyond the rows
    const int q = i * kThreads + (int)threadIdx.x;
    m = kM == 1 ? 0 : q / row_chunks;
    c = q - m * row_chunks;
    return q < all_chunks;
  };
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    int m, c;
    const bool ok = chunk_place(i, m, c) && c * 8 < a.K;
    raw[i] = *reinterpret_cast<const v4u*>(a.X + (ok ? (size_t)m * a.ldx + c * 8 : (size_t)0));
  }
  // the terms of the output that this thread will finish (all threads load, some use it)
  const int tiles = ceil_div(ceil_div(a.N, 16) - (int)blockIdx.x, (int)gridDim.x);   // blockIdx.x, + gridDim.x, ...
  const int out_tile = (int)threadIdx.x / (M * 16), out_m = (int)threadIdx.x % (M * 16) / 16;
  const int out_n = ((int)blockIdx.x + out_tile * (int)gridDim.x) * 16 + lr;
  const bool has_out = out_tile < tiles && out_n < a.N;
  const int safe_n = has_out ? out_n : 0;
  const float out_c = a.c[safe_n];
  const uint16_t* no_term = reinterpret_cast<const uint16_t*>(a.c);   // any address that can be read
  const uint16_t out_bias = *(a.bias ? a.bias + safe_n : no_term);
  const uint16_t out_res = *(a.residual ? a.residual + (size_t)out_m * a.ldr + safe_n : no_term);

  // ---- weights: this wave's slabs of the tiles one after the other
  const int mine = wave < n_slabs ? (n_slabs - wave + WAVES - 1) / WAVES : 0;   // slabs of this wave per tile: at most 64
  const uint32_t lane_off = (lg >> 1) * 1024 + (32 * (lg & 1) + lr) * 16;
  auto tile_base = [&](int t) {
    const int n0 = ((int)blockIdx.x + t * (int)gridDim.x) * 16;
    return a.Wt + (size_t)(n0 >> 8) * n_slabs * kBlockBytes + (size_t)((n0 & 255) >> 5) * 2048 + (n0 & 16) * 16;
  };
  int f_tile = 0, f_slab = 0;                                         // what is requested next; past the end the last slab again
  const int8_t* f_base = tile_base(0);
  auto fetch_w = [&](v4i& w) __attribute__((always_inline)) {
    const int slab = min(wave + WAVES * f_slab, n_slabs - 1);
    w = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(f_base + (size_t)slab * kBlockBytes + lane_off));
    if (f_slab + 1 < mine) {
      ++f_slab;
    } else if (f_tile + 1 < tiles) {
      f_slab = 0;
      f_base = tile_base(++f_tile);
    }
  };
  v4i f[kAhead];
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int i = 0; i < kAhead; ++i) fetch_w(f[i]);
  __builtin_amdgcn_sched_barrier(0);

  for (int t = threadIdx.x; t < n_slabs; t += kThreads) s_any[t] = 0;
  const us2 th2 = __builtin_bit_cast(us2, a.th | (a.th << 16));
  us2 best[kM];
  uint32_t over[kChunks];                                             // bit j: |element j| >= threshold
#pragma unroll
  for (int m = 0; m < kM; ++m) best[m] = __builtin_bit_cast(us2, 0u);
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    int m, c;
    const bool ok = chunk_place(i, m, c) && c * 8 < a.K;              // (the K padding: zeros, never critical)
    us2 t = __builtin_bit_cast(us2, 0u);
    over[i] = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {   // per half, wraps mod 2^16: entries below the threshold get the top bit
      raw[i][w] = ok ? raw[i][w] : 0u;
      const us2 d = (us2)(__builtin_bit_cast(us2, raw[i][w] & 0x7fff7fffu) - th2);
      t = __builtin_elementwise_max(t, d);
      const uint32_t dd = __builtin_bit_cast(uint32_t, d);
      over[i] |= ((~dd >> 15) & 1u) << (2 * w) | ((~dd >> 31) & 1u) << (2 * w + 1);
    }
    if (!ok) over[i] = 0;
#pragma unroll
    for (int mm = 0; mm < kM; ++mm)
      if (ok && mm == m) best[mm] = __builtin_elementwise_max(best[mm], t);
    if constexpr (kM > 1) {
      if (i * kThreads + (int)threadIdx.x < all_chunks) s_over[i * kThreads + threadIdx.x] = (uint8_t)over[i];
    }
  }
#pragma unroll
  for (int m = 0; m < kM; ++m) {
    const uint32_t both = __builtin_bit_cast(uint32_t, best[m]);
    const uint32_t wmax = wave_max_u32(max(both & 0xffffu, both >> 16));
    if (lane == 0) s_part[m][wave] = wmax;
  }
  __syncthreads();
  if ((int)threadIdx.x < M) {
    uint32_t mm = 0;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) mm = max(mm, s_part[threadIdx.x][w]);
    const float r = (mm & 0x8000u) ? half_lo_to_float((mm + a.th) & 0xffffu) : 0.0f;
    s_r[threadIdx.x] = r;
    s_scale[threadIdx.x] = (r == 0.0f) ? 0.0f : 127.0f / r;          // IEEE division
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    // one chunk at a time (bounded registers): the chunk passes through an opaque statement, and such statements keep
    // their order
    asm volatile("" : "+v"(raw[i][0]), "+v"(raw[i][1]), "+v"(raw[i][2]), "+v"(raw[i][3]) : : "memory");
    int m, c;
    if (chunk_place(i, m, c)) {
      const int k = c * 8;
      uint32_t crit = over[i];                                        // bit j: column k + j is critical
      if constexpr (kM > 1) {
#pragma unroll
        for (int mm = 0; mm < kM; ++mm) crit |= mm < M ? s_over[mm * row_chunks + c] : 0u;
      }
      const float sc = s_scale[m];
      uint32_t code[2] = {0, 0}, xf[4];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t h = (raw[i][j >> 1] >> (16 * (j & 1))) & 0xffffu;
        const bool cr = (crit >> j) & 1u;
        code[j >> 2] |= (cr ? 0u : to_code_byte(half_lo_to_float(h), sc)) << (8 * (j & 3));
      }
#pragma unroll
      for (int w = 0; w < 4; ++w)
        xf[w] = (((crit >> (2 * w)) & 1u) ? (raw[i][w] & 0xffffu) : 0u) | (((crit >> (2 * w + 1)) & 1u) ? (raw[i][w] & 0xffff0000u) : 0u);
      *reinterpret_cast<v2u*>(s_code + (size_t)m * Kpad + k) = v2u{code[0], code[1]};
      *reinterpret_cast<v4u*>(s_xf + (size_t)m * Kpad + k) = v4u{xf[0], xf[1], xf[2], xf[3]};
      if (crit) s_any[k >> 6] = 1;
    }
  }
  __syncthreads();

  // ---- the products
  v4i acc = v4i{0, 0, 0, 0};
  v4f accf = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  const bool row_live = lr < M;
  const int row = row_live ? lr : 0;                                  // lanes beyond M read row 0 and feed zeros
  const int8_t* my_code = s_code + (size_t)row * Kpad + lg * 16;
  const uint16_t* my_xf = s_xf + (size_t)row * Kpad + lg * 16;
  // "slab holds a critical column", this wave's slabs
  const uint64_t any_mask = __builtin_amdgcn_ballot_w64(lane < mine && s_any[min(wave + WAVES * lane, n_slabs - 1)] != 0);
  int tile = 0, i_slab = 0;
  // C layout of the 16x16 MFMA: lane = column (lane % 16), register e = row 4 (lane / 16) + e
  auto leave_sums = [&](int t) __attribute__((always_inline)) {
    int32_t* d = s_sum + t * tile_words + wave * M * 16 + lr;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = 4 * lg + e;
      if (m < M) {
        const float sum16 = accf[e];                                  // (a bit cast of a vector's element reads element 0)
        d[m * 16] = acc[e];
        d[(WAVES * M + m) * 16] = __builtin_bit_cast(int32_t, sum16);
      }
    }
    acc = v4i{0, 0, 0, 0};
    accf = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  };
  auto step = [&](v4i& w) __attribute__((always_inline)) {
    const int slab = wave + WAVES * i_slab;
    // lane group lg (0..3) holds columns 16 lg .. + 16 of the slab; the two fp16 instructions take the two
    // halves of every lane group's piece (any split of the 64 columns does, as long as both operands agree)
    v4i xa = *reinterpret_cast<const v4i*>(my_code + slab * kSlabBytes);
    if (!row_live) xa = v4i{0, 0, 0, 0};
    acc = __builtin_amdgcn_mfma_i32_16x16x64_i8(xa, w, acc, 0, 0, 0);
    if ((any_mask >> i_slab) & 1u) {                                  // the same for the whole wave
      const v4u wu = __builtin_bit_cast(v4u, w) ^ 0x80808080u;
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        v4u xr = *reinterpret_cast<const v4u*>(my_xf + slab * kSlabBytes + t * 8);
        if (!row_live) xr = v4u{0, 0, 0, 0};
        accf = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(v8h, xr), codes_to_half8(wu, t), accf, 0, 0, 0);
      }
    }
    fetch_w(w);
    if (++i_slab == mine) {                                           // the tile is done
      leave_sums(tile++);
      i_slab = 0;
    }
  };
  // Whole groups of kAhead slabs run without a way out in between (with an exit after every slab the compiler
  // waited for every request in flight at the end of each group, emptying the queue of weights).
  const int total = tiles * mine;
  int i0 = 0;
  for (; i0 + kAhead <= total; i0 += kAhead) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) step(f[u]);
  }
#pragma unroll
  for (int u = 0; u < kAhead - 1; ++u)
    if (i0 + u < total) step(f[u]);
  if (mine == 0)
    for (int t = 0; t < tiles; ++t) leave_sums(t);                    // (fewer slabs than waves: zeros)
  __syncthreads();

  if (has_out) {
    const int32_t* s = s_sum + out_tile * tile_words + out_m * 16 + lr;
    int32_t sum = 0;
    float sumf = 0.0f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) sum += s[w * M * 16], sumf += __builtin_bit_cast(float, s[(WAVES + w) * M * 16]);
    float y = (float)sum * (s_r[out_m] * (out_c / 16129.0f)) + sumf * (out_c / 127.0f);
    if (a.bias) y += half_lo_to_float(out_bias);
    if (a.lora_r > 0) {                                               // the low-rank term, as k_skinny_finalize adds it
      float low = 0.0f;
      for (int j = 0; j < a.lora_r; j += 8) {
        const v4u t = *reinterpret_cast<const v4u*>(a.lora_T + (size_t)out_m * a.lora_ldt + j);
        const v4u b = *reinterpret_cast<const v4u*>(a.lora_B + (size_t)out_n * a.lora_r + j);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          low += half_lo_to_float(t[e]) * half_lo_to_float(b[e]) + half_hi_to_float(t[e]) * half_hi_to_float(b[e]);
      }
      y += low;
    }
    uint32_t h = float_to_half_bits(y);
    if (a.gelu) h = gelu_to_half_bits(half_lo_to_float(h));
    if (a.residual) h = float_to_half_bits(half_lo_to_float(h) + half_lo_to_float(out_res));
    a.Y[(size_t)out_m * a.ldy + out_n] = (uint16_t)h;
    if (a.tap_acc) a.tap_acc[(size_t)out_m * a.N + out_n] = sum;
  }
}

constexpr int kRowsMaxChunks = 6;   // of the largest instantiation

// dynamic LDS of a call whose workgroups have `tiles` tiles each
static size_t rows_lds_bytes(int M, int Kpad, int tiles) {
  return (size_t)3 * M * Kpad + (M > 1 ? round_up(M * Kpad / 8, 16) : 0) + (size_t)tiles * 2 * kRowsWaves * M * 16 * 4;
}
// most tiles a workgroup can have: their sums in LDS, an output per thread
static int rows_tiles_max(int M, int Kpad) {
  const long room = (long)kRowsMaxLds - (long)rows_lds_bytes(M, Kpad, 0);
  return room <= 0 ? 0 : (int)min(room / (2 * kRowsWaves * M * 16 * 4), (long)(kRowsWaves * kWave / (16 * M)));
}
// Up to four rows wherever they fit in LDS; more where a compute unit can hold the sums of all its tiles, so that it
// prepares once (six rows of a 7B layer 67 us, 74 with K split between workgroups; eight rows, where 4096 x 22016 prepares
// twice, 38 us for that linear, 31 split).
bool rows_kernel_fits(int M, int Kpad, int N) {
  return M >= 1 && M <= kRowsMaxM && M * Kpad / 8 <= kRowsMaxChunks * kRowsWaves * kWave &&
         rows_tiles_max(M, Kpad) >= (M <= 4 ? 1 : ceil_div(ceil_div(N, 16), device_cu_count()));
}

// more than the default 64 KB of LDS: an attribute per kernel and device
template <int kM, int... kChunks>
static hipError_t prepare_rows_of() {
  for (const void* fn : {reinterpret_cast<const void*>(&k_gemm_rows<kM, kChunks>)...})
    if (hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kRowsMaxLds); e != hipSuccess) return e;
  return hipSuccess;
}
hipError_t prepare_rows_kernels() {
  static std::atomic<bool> attr_set[64] = {};                      // setting an attribute twice is harmless
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (attr_set[dev]) return hipSuccess;
  hipError_t e = prepare_rows_of<1, 1, 2, 3, kRowsMaxChunks>();
  if (e == hipSuccess) e = prepare_rows_of<2, 1, 2, 3, kRowsMaxChunks>();
  if (e == hipSuccess) e = prepare_rows_of<4, 1, 2, 3, kRowsMaxChunks>();
  if (e == hipSuccess) e = prepare_rows_of<8, 1, 2, 3, kRowsMaxChunks>();
  if (e == hipSuccess) attr_set[dev] = true;
  return e;
}

template <int kM>
static hipError_t launch_rows_of(const SkinnyArgs& a, int chunks, int grid, size_t lds, hipStream_t stream) {
  const dim3 g(grid), b(kRowsWaves * kWave);
  if (chunks <= 1) hipLaunchKernelGGL((k_gemm_rows<kM, 1>), g, b, lds, stream, a);
  else if (chunks <= 2) hipLaunchKernelGGL((k_gemm_rows<kM, 2>), g, b, lds, stream, a);
  else if (chunks <= 3) hipLaunchKernelGGL((k_gemm_rows<kM, 3>), g, b, lds, stream, a);
  else hipLaunchKernelGGL((k_gemm_rows<kM, kRowsMaxChunks>), g, b, lds, stream, a);
  return hipGetLastError();
}

hipError_t launch_gemm_rows(SkinnyArgs a, hipStream_t stream) {
  a.n_slabs = packed_k(a.K) / kSlabBytes;
  const int Kpad = a.n_slabs * kSlabBytes;
  if (!a.X || !rows_kernel_fits(a.M, Kpad, a.N) || a.codes) return hipErrorInvalidValue;
  if (hipError_t e = prepare_rows_kernels(); e != hipSuccess) return e;
  // a workgroup per compute unit, its tiles one after the other; more workgroups where their sums would not fit in LDS
  const int n_tiles = ceil_div(a.N, 16), per = min(ceil_div(n_tiles, device_cu_count()), rows_tiles_max(a.M, Kpad));
  const int grid = per == ceil_div(n_tiles, device_cu_count()) ? min(n_tiles, device_cu_count()) : ceil_div(n_tiles, per);
  const size_t lds = rows_lds_bytes(a.M, Kpad, ceil_div(n_tiles, grid));
  const int chunks = ceil_div(a.M * Kpad / 8, kRowsWaves * kWave);
  if (a.M == 1) return launch_rows_of<1>(a, chunks, grid, lds, stream);
  if (a.M == 2) return launch_rows_of<2>(a, chunks, grid, lds, stream);
  if (a.M <= 4) return launch_rows_of<4>(a, chunks, grid, lds, stream);
  return launch_rows_of<8>(a, chunks, grid, lds, stream);
}

}  // namespace mmd8
