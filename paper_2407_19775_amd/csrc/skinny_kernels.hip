// Decode-shaped (at most 128 tokens) mixed int8 GEMM ("Compression techniques", item 2): bound by
// streaming the int8 weights once from HBM, not by the matrix pipes.
//
//   acc[m,n] = sum_k Xq[m,k] Wt[n,k]                                   int8 MFMA, exact
//   Y[m,n]   = f16( acc r[m] c[n] / 127^2 + sum_{k critical} X[m,k] f16(Wt[n,k] c[n]/127) + bias[n] )
//
// Heavy-tailed decode activations flag a large share of the feature dimensions, so the 16-bit part
// is a second product over the same weights rather than a small correction.
// To keep the conversion of the weights cheap the fp16 operand is the integer code itself (exact
// in fp16, one byte permute and one packed fp16 subtraction per two codes) and the column step
// c[n]/127 is applied in fp32 to the accumulated sum: the sum over the critical columns of
// X[m,k] q[n,k] c[n]/127 with one rounding at the end, instead of rounding each dequantized weight
// to fp16 first.  The two differ by at most the fp16 rounding of the weights (2^-11 relative per
// term), far inside the tolerance of the fp16 output.
#include <math.h>

#include <type_traits>
#include <utility>

#include <atomic>

#include "codec_device.h"
#include "common.h"
#include "operand_layout.h"
#include "skinny.h"

namespace mmd8 {

typedef short ss2 __attribute__((ext_vector_type(2)));

// ------------------------------------------------------------------------------------------------
// A workgroup of eight waves multiplies up to kBM rows with one 256-column weight panel over a range of K, 64 columns of K
// (a slab) at a time.  Everything of a slab comes through one ring of LDS buffers by global_load_lds_dwordx4: the
// activation codes, the rows of X themselves (128 bytes per row, eight rows per request) and the weight codes.  Which
// columns are critical is decided on the weight side: a weight code goes into the int8 product where its column is not
// critical and into the fp16 product, as an integer, where it is (masks of 256 slabs at a time in LDS, a byte per column), so
// the preparation need not know the critical columns when it writes the codes: one pass over X, no fp16 copy.  (Entries of
// other columns are below the threshold, hence finite, and so is what stands in for the padding of K: zero times them is zero.)
// A wave owns 64 columns: of all rows and one of the slab's two k-steps (up to 64 rows; the two halves are added in
// LDS at the end), or of 64 rows and both k-steps (128 rows).  64 x 64 accumulators per wave keep the LDS reads below what
// the fills take: with 32 columns per wave a slab's activation side was read twice as often, and 64 rows took 0.8 us per slab.
// The ranges leave fp32 sums, added in a fixed order by a second kernel (the result does not depend on timing).
//
// What bounds it: a compute unit takes in about 57 bytes per ns where part of them comes from memory (its loads come back
// in order), and a slab is 22 (32 rows), 28 (64) or 40 KB (128) for 16 KB of weights; 16 KB for every compute unit take
// 0.65 us from HBM.  Measured on 4096 -> 22016 (172 workgroups of 32 slabs): 0.49, 0.65 and 1.1 us per slab, and before the
// first and after the last of them 3 us (0.7 addresses, 2 first bytes from memory) and 1.6 to 3.5 us (sums to memory).  The
// weights are requested as bytes that nothing else reads: with the plain request a 7B layer takes 95.8 instead of 87.3 us
// at 32 rows.  Whole layers of that shape, weights from memory, where scan, pack and a kernel with the weights straight in
// registers took (two passes of it for more than 64 rows): 16 rows 96 -> 79 us, 32 rows 98 -> 86, 64 rows 132 -> 109, 100
// rows 246 -> 146, 128 rows 261 -> 156; of 70B shape 32 rows 214 -> 200, 128 rows 491 -> 392.
// ------------------------------------------------------------------------------------------------
template <int kBM_>
struct DecodeCfg {
  static constexpr int kBM = kBM_, kWaves = 8, kThreads = kWaves * kWave;
  static constexpr bool kHalves = kBM <= 64;                         // the waves 4..7 take the second k-step of every slab
  static constexpr int TI = kBM == 32 ? 1 : 2, TJ = 2;               // 32 x 32 tiles of a wave
  static constexpr int kCodes = kBM * kSlabBytes, kRows = 2 * kCodes, kStage = kCodes + kRows + kBlockBytes;
  static constexpr int kStages = kBM == 32 ? 5 : kBM == 64 ? 4 : 3;
  static constexpr int kPieces = kStage / 1024;                      // 1 KB requests per slab
  static constexpr int kReq = (kPieces + kWaves - 1) / kWaves;       // per wave; the waves from kFullWaves on make one less
  static constexpr int kFullWaves = kPieces - kWaves * (kReq - 1);
  static constexpr int kMaskSlabs = 256;
  static constexpr int kMaskAt = kStages * kStage, kScalesAt = kMaskAt + kMaskSlabs * kSlabBytes;
  static constexpr int LDS_BYTES = kScalesAt + 4 * kBM;
  static_assert(LDS_BYTES <= 160 * 1024 && kScalesAt >= (kHalves ? 2 : 1) * kBM * 1024, "LDS, which also takes the sums");
  static_assert((kStages - 1) * kReq <= 63, "requests in flight fit the wait instruction's count");
};

// own requests are in but the newest kVm, own LDS reads have returned
template <int kVm>
__device__ __forceinline__ void wait_requests() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(kVm) : "memory");
}

template <int kBM>
__global__ __launch_bounds__(DecodeCfg<kBM>::kThreads) void k_gemm_decode(const SkinnyArgs a) {
  using Cfg = DecodeCfg<kBM>;
  constexpr int TI = Cfg::TI, TJ = Cfg::TJ, kStages = Cfg::kStages, kReq = Cfg::kReq;
  extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
  int8_t* s_mask = smem + Cfg::kMaskAt;
  float* s_r = reinterpret_cast<float*>(smem + Cfg::kScalesAt);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lr = lane & 31, lg = lane >> 5;
  const int half = wave >> 2, wn = wave & 3;                         // half: k-step of the slab, or 64-row half of the tile
  const int tile = blockIdx.x % a.tiles_n, split = blockIdx.x / a.tiles_n;
  const int first = split * a.slabs_per_split, end = min(first + a.slabs_per_split, a.n_slabs), last = end - 1;
  const int n0 = tile * 256 + wn * 64;

  // ---- what is not part of the stream, asked for ahead of it: the terms of this wave's columns and of the rows (for the
  // end), and the column flags of the range, copied to LDS where they become masks
  float c[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) c[j] = a.c[min(n0 + j * 32 + lr, a.N - 1)];
  const float r0 = a.r[min((int)threadIdx.x, a.M - 1)];
  auto mask_words = [&](int s0) { return min(Cfg::kMaskSlabs, end - s0) * (kSlabBytes / 4); };
  auto put_mask = [&](int t, uint32_t flags) {                       // 4 columns
    flags &= 0x01010101u;
    reinterpret_cast<uint32_t*>(s_mask)[t] = flags * 0xffu;
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  __builtin_amdgcn_sched_barrier(0);
  // (whole KB, up to 15 slabs past the range: still inside the workspace)
  for (int i = wave; 1024 * i < 4 * mask_words(first); i += Cfg::kWaves)
    dma16(a.mask + (size_t)first * kSlabBytes + i * 1024 + lane * 16, lds0 + Cfg::kMaskAt + i * 1024);

  // ---- requests: piece 8 d + wave of a slab's 1 KB pieces, codes first, then rows, then weights
  const bool full_wave = wave < Cfg::kFullWaves;
  const int whole_slabs = a.K / kSlabBytes;
  const int8_t* src[kReq];                                            // of the slab that is requested next
  int step[kReq];                                                     // bytes from a slab to the next
  int row_piece[kReq];                                                // first column of this lane's 16 bytes of a row of X
#pragma unroll
  for (int d = 0; d < kReq; ++d) {
    const int i = min(8 * d + wave, Cfg::kPieces - 1);
    step[d] = kBlockBytes;
    row_piece[d] = 0;
    if (i < Cfg::kCodes / 1024) {
      src[d] = a.Xq + i * 1024 + lane * 16;
    } else if (i < (Cfg::kCodes + Cfg::kRows) / 1024) {
      // row R keeps its 16-byte piece q at place q ^ (R / 2 % 8): 16 lanes of a fragment read meet every bank once
      const int row = 8 * (i - Cfg::kCodes / 1024) + (lane >> 3);
      row_piece[d] = 8 * ((lane & 7) ^ (row >> 1 & 7));
      step[d] = 2 * kSlabBytes;
      src[d] = reinterpret_cast<const int8_t*>(a.X + (size_t)min(row, a.M - 1) * a.ldx + row_piece[d]);
    } else {
      src[d] = a.Wt + (size_t)tile * a.n_slabs * kBlockBytes + (i - (Cfg::kCodes + Cfg::kRows) / 1024) * 1024 + lane * 16;
    }
    src[d] += (size_t)first * step[d];
  }
  auto request = [&](int s, int stage, int d, auto whole_tag) __attribute__((always_inline)) {
    const int8_t* p = src[d];
    if (!decltype(whole_tag)::value && s >= whole_slabs && step[d] != kBlockBytes) {
      // columns beyond K (a multiple of 16): column flags in their place, as halves finite numbers; their weights are zero
      // (entries of X would not do: a critical one may be infinite)
      if (s * kSlabBytes + row_piece[d] >= a.K) p = reinterpret_cast<const int8_t*>(a.mask);
    }
    const uint32_t dst = lds0 + stage * Cfg::kStage + (8 * d + wave) * 1024;
    if (8 * d * 1024 >= Cfg::kCodes + Cfg::kRows) dma16_once(p, dst);   // (weights, whichever wave)
    else dma16(p, dst);
    src[d] += step[d];
  };
  auto request_slab = [&](int s, int stage) __attribute__((always_inline)) {
#pragma unroll
    for (int d = 0; d < kReq; ++d)
      if (d + 1 < kReq || full_wave) request(s, stage, d, std::false_type{});
  };
  // own requests are in but those of the newest `behind` slabs (at most kStages - 1), own LDS reads have returned; then a
  // barrier: the same holds for every wave
  auto wait_for = [&](int behind) __attribute__((always_inline)) {
    // (the usual count first)
    auto wait = [&]<int... kB>(std::integer_sequence<int, kB...>, auto req_tag) __attribute__((always_inline)) {
      (void)((behind == kStages - 1 - kB ? (wait_requests<(kStages - 1 - kB) * decltype(req_tag)::value>(), true) : false) || ...);
    };
    if (full_wave) wait(std::make_integer_sequence<int, kStages>{}, std::integral_constant<int, kReq>{});
    else wait(std::make_integer_sequence<int, kStages>{}, std::integral_constant<int, kReq - 1>{});
    asm volatile("s_barrier" : : : "memory");
  };

  // ---- fragments of one k-step
  struct Frags {
    v4i x[TI], w[TJ];        // codes of both sides
    v4u xf[2][TI], mk;       // rows of X, the two halves of the k-step; 0xff per critical column
  };
  const int row_group = Cfg::kHalves ? 0 : 2 * half;                  // first 32-row group of this wave
  const int a_off = row_group * 2048 + lane * 16;
  const int b_off = Cfg::kCodes + Cfg::kRows + wn * 4096 + lane * 16;
  const int x_off = Cfg::kCodes + (row_group * 32 + lr) * (2 * kSlabBytes);
  constexpr int kReads = TI + TJ + 1 + 2 * TI;
  auto read_frag = [&](int s, int stage, int ks, Frags& f, int n) __attribute__((always_inline)) {
    const int8_t* base = smem + stage * Cfg::kStage;
    if (n < TJ)
      f.w[n] = *reinterpret_cast<const v4i*>(base + b_off + n * 2048 + ks * 1024);
    else if (n == TJ)
      f.mk = *reinterpret_cast<const v4u*>(s_mask + ((s - first) & (Cfg::kMaskSlabs - 1)) * kSlabBytes + (2 * ks + lg) * 16);
    else if (n < TJ + 1 + TI)
      f.x[n - TJ - 1] = *reinterpret_cast<const v4i*>(base + a_off + (n - TJ - 1) * 2048 + ks * 1024);
    else {
      const int t = (n - TJ - 1 - TI) / TI, i = (n - TJ - 1 - TI) % TI;
      const int q = 4 * ks + 2 * lg + t;                              // columns 8 q .. 8 q + 8 of the slab
      f.xf[t][i] = *reinterpret_cast<const v4u*>(base + x_off + i * (32 * 2 * kSlabBytes) + ((q ^ (lr >> 1 & 7)) * 16));
    }
  };

  v16i acc[TI][TJ];
  v16f accf[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0, accf[i][j][e] = 0.0f;

  // The products of one k-step.  Between any two MFMAs `between(n)` (a fragment read of the next k-step, at times a
  // request) and the conversion of weight codes ahead of their MFMA, fenced so that they stay there: a wave issues in
  // order, and a burst of reads that finds the LDS queue full holds up the MFMAs behind it.
  constexpr int kInt = TI * TJ, kAll = 3 * kInt;
  auto multiply = [&](const Frags& g, auto&& between) __attribute__((always_inline)) {
    v2u wh[2 * TJ][2];
    v4i wi[TJ];
#pragma unroll
    for (int n = 0; n < kAll; ++n) {
      if (n < kInt) {
        const int i = n % TI, j = n / TI;
        if (i == 0) wi[j] = __builtin_bit_cast(v4i, __builtin_bit_cast(v4u, g.w[j]) & ~g.mk);
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(g.x[i], wi[j], acc[i][j], 0, 0, 0);
      } else {
        const int q = (n - kInt) / TI, t = q / TJ, j = q % TJ, i = n % TI;
        const v4u h = v4u{wh[q][0][0], wh[q][0][1], wh[q][1][0], wh[q][1][1]};
        accf[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, g.xf[t][i]), __builtin_bit_cast(v8h, h), accf[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      between(n);
      // (word d of conversion q, kInt MFMAs ahead of its own)
#pragma unroll
      for (int w = 0; w < 2 / TI; ++w) {
        const int x = n * (2 / TI) + w, q = x >> 1, t = q / TJ, j = q % TJ, d = x & 1;
        if (q < 2 * TJ) wh[q][d] = codes_to_half4(((uint32_t)g.w[j][2 * t + d] & g.mk[2 * t + d]) ^ 0x80808080u);   // other columns: zero
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

#pragma unroll
  for (int q = 0; q < kStages; ++q)
    if (first + q < end) request_slab(first + q, q);
  Frags f[2];
  wait_for(min(kStages - 1, last - first));                           // slab `first` has landed, and the flags
  for (int t = threadIdx.x; t < mask_words(first); t += Cfg::kThreads) put_mask(t, reinterpret_cast<const uint32_t*>(s_mask)[t]);
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" : : : "memory");
  const int ks0 = Cfg::kHalves ? half : 0;
#pragma unroll
  for (int n = 0; n < kReads; ++n) read_frag(first, 0, ks0, f[0], n);
  int stage = 0, s = first;
  // Slab s (the fragments of its first k-step are in g): once slab s + 1 has landed everywhere, its fragments are read
  // into `next` between the MFMAs, and slab s + kStages is requested into the buffer of slab s, whose fragments every
  // wave has read by then.  steady: all of that is there, and within K.
  auto slab = [&](Frags& g, Frags& next, auto steady_tag) __attribute__((always_inline)) {
    constexpr bool kSteady = decltype(steady_tag)::value;
    const int stage1 = stage + 1 == kStages ? 0 : stage + 1;
    if constexpr (!Cfg::kHalves) {                                     // the second k-step of this slab
      multiply(g, [&](int n) __attribute__((always_inline)) {
        if (n < kReads) read_frag(s, stage, 1, next, n);
      });
    }
    const bool ask = kSteady || s + kStages <= last;
    if constexpr (kSteady) {
      if (full_wave) wait_requests<(kStages - 2) * kReq>();
      else wait_requests<(kStages - 2) * (kReq - 1)>();
      asm volatile("s_barrier" : : : "memory");
    } else if (s < last) {
      wait_for(min(kStages - 2, last - s - 1));
    }
    Frags& from = Cfg::kHalves ? g : next;
    Frags& to = Cfg::kHalves ? next : g;
    // (past the end the fragments read are those of an older slab, and not used)
    multiply(from, [&](int n) __attribute__((always_inline)) {
      if (n < kReads) read_frag(s + 1, stage1, ks0, to, n);
      const int d = n * kReq / kAll;
      if (d < kReq && (d * kAll + kReq - 1) / kReq == n && ask && (d + 1 < kReq || full_wave)) request(s + kStages, stage, d, steady_tag);
    });
    stage = stage1;
    ++s;
  };
  // (A short range runs the general form of the loop only: what is entered first has to be fetched as instructions.  With the
  // steady form for every range 4096 -> 4096 took 12.3 us at 32 rows instead of 10.8, with the general form for every
  // range 4096 -> 22016 25.2 instead of 23.2.)
  const int steady_end = end - first >= 20 ? min(last, whole_slabs - 1) - kStages : first;
  for (int window = first;; window += Cfg::kMaskSlabs) {
    const int to = min(window + Cfg::kMaskSlabs, end);                 // (an even number of slabs but for the last window)
    while (s < min(to, steady_end)) {                                  // (an even number of slabs)
      slab(f[0], f[1], std::true_type{});
      if constexpr (Cfg::kHalves) slab(f[1], f[0], std::true_type{});
    }
    while (s < to) {
      slab(f[0], f[1], std::false_type{});
      if constexpr (Cfg::kHalves) {
        if (s < to) slab(f[1], f[0], std::false_type{});
      }
    }
    if (to == end) break;
    __syncthreads();                                                   // every wave has read the masks so far
    for (int t = threadIdx.x; t < mask_words(to); t += Cfg::kThreads)
      put_mask(t, reinterpret_cast<const uint32_t*>(a.mask + (size_t)to * kSlabBytes)[t]);
    __syncthreads();
    read_frag(s, stage, ks0, f[0], TJ);                                // the mask of slab s again
  }

  // ---- the sums of this range, through LDS: as fp32 rows of 256 columns (of either half of the slabs), then in a loop whole
  // rows to memory.  (This code runs once and is not in the instruction cache when it is reached: what counts is how
  // little of it there is.  With the halves exchanged register by register and every element stored from its own register
  // it took 2.7 us at 32 rows and 4.6 at 64.)
  // C layout of the 32x32 MFMA: lane = column (lane % 32), register e = row 8 (e / 4) + 4 (lane / 32) + (e % 4); the rows
  // of the upper lanes swap the two 32-column halves of every 64 (the other 32 banks).
  if ((int)threadIdx.x < kBM) s_r[threadIdx.x] = r0;
  __syncthreads();
  float* s_y = reinterpret_cast<float*>(smem);                        // [half][kBM][256]
#pragma unroll
  for (int j = 0; j < TJ; ++j) {
    const float cs = c[j] / 16129.0f, col_step = c[j] / 127.0f;
    float* const mine = s_y + ((Cfg::kHalves ? half * kBM : row_group * 32) + 4 * lg) * 256 + wn * 64 + ((j ^ lg) * 32 + lr);
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const v4f rm = *reinterpret_cast<const v4f*>(s_r + (row_group + i) * 32 + 8 * q + 4 * lg);
#pragma unroll
        for (int e = 0; e < 4; ++e) mine[(i * 32 + 8 * q + e) * 256] = (float)acc[i][j][4 * q + e] * (rm[e] * cs) + accf[i][j][4 * q + e] * col_step;
      }
  }
  if (a.tap_acc) {                                                   // (zeroed by the launcher; integers, so in any order)
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int m = (row_group + i) * 32 + 8 * (e >> 2) + 4 * lg + (e & 3), n = n0 + j * 32 + lr;
          if (m < a.M && n < a.N) atomicAdd(a.tap_acc + (size_t)m * a.N + n, acc[i][j][e]);
        }
  }
  __syncthreads();
  const int col = 4 * lane, n = tile * 256 + col;                     // a wave per row
  if (n >= a.N) return;
  float* dst = a.partial + (size_t)split * a.M * a.N + n;
  for (int m = wave; m < a.M; m += Cfg::kWaves) {
    const float* y = s_y + m * 256 + (col ^ ((m & 4) * 8));
    v4f v = *reinterpret_cast<const v4f*>(y);
    if constexpr (Cfg::kHalves) v += *reinterpret_cast<const v4f*>(y + kBM * 256);
    *reinterpret_cast<v4f*>(dst + (size_t)m * a.N) = v;
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
// order, then the bias, then the low-rank term (T as sums P of ranges, B: [N][r] fp16, r a multiple of 8;
// r == 0: no such term).  A row per blockIdx.y.
__global__ __launch_bounds__(256) void k_skinny_finalize(const float* __restrict__ partial, int splits, int M, int N,
                                                         const uint16_t* __restrict__ bias,
                                                         const float* __restrict__ P, int p_splits,
                                                         const uint16_t* __restrict__ B, int r, uint16_t* __restrict__ T_user,
                                                         const uint16_t* residual /* may alias Y */, int ldr, int gelu,
                                                         uint16_t* Y, int ldy, uint8_t* flag_reset, int Kpad) {
  if (blockIdx.y == 0) reset_column_flags(flag_reset, Kpad);
  const int m = blockIdx.y, n = (int)blockIdx.x * 256 + (int)threadIdx.x;
  __shared__ __attribute__((aligned(16))) uint16_t s_T[kLoraMaxRank];
  if (r > 0) {                                                       // this row of T
    if ((int)threadIdx.x < r) {
      const uint32_t t = sum_low_rank_activation(P, p_splits, M, m, threadIdx.x);
      s_T[threadIdx.x] = (uint16_t)t;
      if (T_user && blockIdx.x == 0) T_user[(size_t)m * r + threadIdx.x] = (uint16_t)t;
    }
    __syncthreads();
  }
  if (n >= N) return;
  // Asked for ahead of the sums and whether there or not (a dword of the sums in their place): behind the sums, under a
  // condition, the residual was one more memory latency.
  const uint16_t* at = reinterpret_cast<const uint16_t*>(partial + (size_t)m * N + n);
  const uint16_t bias_n = *(bias ? bias + n : at), residual_n = *(residual ? residual + (size_t)m * ldr + n : at);
  __builtin_amdgcn_sched_barrier(0);
  float sum[1];
  add_ranges<1>(partial + (size_t)m * N + n, splits, (size_t)M * N, sum);
  float y = sum[0];
  if (bias) y += half_lo_to_float(bias_n);
  if (r > 0) {
    float low = 0.0f;
    for (int j = 0; j < r; j += 8) {
      const v4u t = *reinterpret_cast<const v4u*>(s_T + j);
      const v4u b = *reinterpret_cast<const v4u*>(B + (size_t)n * r + j);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        low += half_lo_to_float(t[e]) * half_lo_to_float(b[e]) + half_hi_to_float(t[e]) * half_hi_to_float(b[e]);
    }
    y += low;
  }
  uint32_t h = float_to_half_bits(y);
  if (gelu) h = gelu_to_half_bits(half_lo_to_float(h));
  if (residual) h = float_to_half_bits(half_lo_to_float(h) + half_lo_to_float(residual_n));
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
  // (ahead of the sums, as in k_skinny_finalize)
  const uint16_t* at = reinterpret_cast<const uint16_t*>(a.partial + (size_t)m * a.N + n);
  const uint16_t* bias_at = a.bias ? a.bias + n : at;                 // (halves: a bias need not be aligned to more)
  const v2u res = *reinterpret_cast<const v2u*>(a.residual ? a.residual + (size_t)m * a.ldr + n : at);
  uint16_t bias[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) bias[i] = bias_at[i];
  __builtin_amdgcn_sched_barrier(0);
  float y[4];
  add_ranges<4>(a.partial + (size_t)m * a.N + n, a.splits, (size_t)a.M * a.N, y);
  uint32_t h[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    h[i] = float_to_half_bits(a.bias ? y[i] + half_lo_to_float(bias[i]) : y[i]);
    if (a.gelu) h[i] = gelu_to_half_bits(half_lo_to_float(h[i]));
  }
  if (a.residual) {
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

// ------------------------------------------------------------------------------------------------
// A few rows whose operands do not fit in LDS (k_gemm_rows below): the eight waves of a workgroup own neighbouring 32-column
// groups of a weight panel and walk a range of K together, weights straight from memory into the registers of the lane that
// feeds them to the MFMA, three slabs ahead.  The activation side is made here: every workgroup streams the rows of X once for
// the row scales, keeps the columns of its own range in LDS with one "critical" flag per column, and writes the codes and the
// fp16 critical columns of a slab into a ring two slabs ahead of the MFMAs: wave w owns the 16-column piece w % 4 of the slab,
// a lane one column of one of four rows.  Rows of the ring beyond M are zeroed once and never written.  With K in one range and
// nothing behind the bias this is the whole layer.
//
// What bounds it: the rows through every compute unit ahead of the first product, and a barrier per slab.  What it saves
// against k_prep_rows and k_gemm_decode is a launch, with K in one range two (plan_panel has both sides measured).
// ------------------------------------------------------------------------------------------------
constexpr int kPanelWaves = 8, kPanelThreads = kPanelWaves * kWave;
constexpr int kPanelMaxSlabs = 128, kPanelMaxRowSlabs = 256;   // of a workgroup's range: its columns of X and their flags in LDS
template <bool kSplit, bool kTap>
__global__ __launch_bounds__(kPanelThreads, 2) void k_gemm_panel(const SkinnyArgs a) {
  constexpr int kThreads = kPanelThreads, kCodes = 2048, kStage = kCodes + 4096;   // of a slab in the ring: 32 rows of codes, then of halves
  __shared__ __attribute__((aligned(16))) int8_t s_x[4][kStage];
  __shared__ uint8_t s_any[kPanelMaxSlabs];
  __shared__ __attribute__((aligned(16))) uint16_t s_row[kPanelMaxRowSlabs * kSlabBytes];   // [M][cnt x 64]
  __shared__ __attribute__((aligned(16))) uint8_t s_crit[kPanelMaxSlabs * kSlabBytes];      // [cnt x 64]
  __shared__ uint32_t s_part[kPanelMaxM][kPanelWaves];
  __shared__ float s_r[kPanelMaxM], s_scale[kPanelMaxM];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int lr = lane & 31, lg = lane >> 5;
  reset_column_flags(a.flag_reset, a.Kpad);
  const int tile = blockIdx.x % a.tiles_n, split = blockIdx.x / a.tiles_n;
  const int n0 = tile * 256 + wave * 32;                              // < Npad: the padding rows of Wt are zero
  const int n = n0 + lr;
  const int s_begin = split * a.slabs_per_split;
  const int cnt = min(a.n_slabs, s_begin + a.slabs_per_split) - s_begin;   // >= 1 by construction of the plan
  const int last = cnt - 1;
  const int8_t* wgrp = a.Wt + (size_t)tile * a.n_slabs * kBlockBytes + (size_t)wave * 2048 + lane * 16 + (size_t)s_begin * kBlockBytes;

  struct Weights {
    v4i w[2];
  };
  auto fetch_w = [&](int j, Weights& f) {
    const int8_t* p = wgrp + (size_t)j * kBlockBytes;
    f.w[0] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p));
    f.w[1] = __builtin_nontemporal_load(reinterpret_cast<const v4i*>(p + 1024));
  };
  Weights f[4];
  fetch_w(0, f[0]);
  fetch_w(min(1, last), f[1]);
  fetch_w(min(2, last), f[2]);

  // ---- scales, columns of the range, their flags (the weight requests above are in flight meanwhile)
  for (int i = threadIdx.x; i < 4 * kStage / 16; i += kThreads) reinterpret_cast<v4u*>(&s_x[0][0])[i] = v4u{0, 0, 0, 0};
  const us2 th2 = __builtin_bit_cast(us2, a.th | (a.th << 16));
  us2 best[kPanelMaxM];
#pragma unroll
  for (int m = 0; m < kPanelMaxM; ++m) best[m] = __builtin_bit_cast(us2, 0u);
  // (rows innermost, so that the loads of all rows are in flight together)
  for (int c = threadIdx.x; c < a.K / 8; c += kThreads) {
    v4u raw[kPanelMaxM];
#pragma unroll
    for (int m = 0; m < kPanelMaxM; ++m) {
      raw[m] = v4u{0, 0, 0, 0};
      if (m < a.M) raw[m] = *reinterpret_cast<const v4u*>(a.X + (size_t)m * a.ldx + c * 8);
    }
#pragma unroll
    for (int m = 0; m < kPanelMaxM; ++m)
#pragma unroll
      for (int w = 0; w < 4; ++w)   // per half, wraps mod 2^16: entries below the threshold get the top bit
        best[m] = __builtin_elementwise_max(best[m], (us2)(__builtin_bit_cast(us2, raw[m][w] & 0x7fff7fffu) - th2));
  }
  const int row_stride = cnt * kSlabBytes;                            // elements of s_row per row
  for (int c = threadIdx.x; c < cnt * (kSlabBytes / 8); c += kThreads) {
    const int k = s_begin * kSlabBytes + c * 8;                       // (the K padding reads as zero)
    v4u raw[kPanelMaxM];
#pragma unroll
    for (int m = 0; m < kPanelMaxM; ++m) {
      raw[m] = v4u{0, 0, 0, 0};
      if (m < a.M && k < a.K) raw[m] = *reinterpret_cast<const v4u*>(a.X + (size_t)m * a.ldx + k);
    }
#pragma unroll
    for (int m = 0; m < kPanelMaxM; ++m)
      if (m < a.M) *reinterpret_cast<v4u*>(&s_row[m * row_stride + c * 8]) = raw[m];
  }
#pragma unroll
  for (int m = 0; m < kPanelMaxM; ++m) {
    if (m < a.M) {                                                    // the same for every lane
      const uint32_t both = __builtin_bit_cast(uint32_t, best[m]);
      const uint32_t wmax = wave_max_u32(max(both & 0xffffu, both >> 16));
      if (lane == 0) s_part[m][wave] = wmax;
    }
  }
  __syncthreads();
  for (int c = threadIdx.x; c < row_stride; c += kThreads) {
    bool crit = false;
    for (int m = 0; m < a.M; ++m) crit = crit || (s_row[m * row_stride + c] & 0x7fffu) >= a.th;
    s_crit[c] = crit ? 1 : 0;
  }
  if ((int)threadIdx.x < a.M) {
    uint32_t mm = 0;
#pragma unroll
    for (int w = 0; w < kPanelWaves; ++w) mm = max(mm, s_part[threadIdx.x][w]);
    // top bit set: an entry below the threshold exists and its pattern is mm + th (mod 2^16)
    const float r = (mm & 0x8000u) ? half_lo_to_float((mm + a.th) & 0xffffu) : 0.0f;
    s_r[threadIdx.x] = r;
    s_scale[threadIdx.x] = (r == 0.0f) ? 0.0f : 127.0f / r;           // IEEE division
  }
  __syncthreads();
  for (int t = threadIdx.x; t < cnt; t += kThreads) {                 // "slab t holds a critical column"
    const v4u* fl = reinterpret_cast<const v4u*>(&s_crit[t * kSlabBytes]);
    const v4u m = fl[0] | fl[1] | fl[2] | fl[3];
    s_any[t] = (m[0] | m[1] | m[2] | m[3]) != 0;
  }

  // slab j of the range -> ring buffer `stage`
  auto make_slab = [&](int j, int stage) {
    const int ch = wave & 3, ks = ch >> 1, g = ch & 1, col = lane & 15;
    const int kl = j * kSlabBytes + ch * 16 + col;
    const bool crit = s_crit[kl] != 0;
    for (int m = (wave >> 2) * 4 + (lane >> 4); m < a.M; m += kPanelWaves) {
      const uint32_t x = s_row[m * row_stride + kl];
      const uint32_t code = crit ? 0u : to_code_byte(half_lo_to_float(x), s_scale[m]);
      s_x[stage][ks * 1024 + (32 * g + m) * 16 + col] = (int8_t)code;
      *reinterpret_cast<uint16_t*>(&s_x[stage][kCodes + (2 * ks + (col >> 3)) * 1024 + (32 * g + m) * 16 + (col & 7) * 2]) =
          crit ? (uint16_t)x : (uint16_t)0;
    }
  };
  struct Frags {
    v4i x[2];      // int8 codes, k-steps 0 and 1
    v8h xf[4];     // fp16 critical columns, pieces 2 (k-step) + t (valid when the slab has any)
  };
  auto read_frags = [&](int stage, bool any, Frags& g) {
    const int8_t* base = &s_x[stage][lane * 16];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) g.x[ks] = *reinterpret_cast<const v4i*>(base + ks * 1024);
    if (any) {                                                        // the same for the whole workgroup
#pragma unroll
      for (int p = 0; p < 4; ++p) g.xf[p] = *reinterpret_cast<const v8h*>(base + kCodes + p * 1024);
    }
  };
  v16i acc;
  v16f accf;
#pragma unroll
  for (int e = 0; e < 16; ++e) acc[e] = 0, accf[e] = 0.0f;
  auto multiply = [&](bool any, const Frags& g, const Weights& w) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) acc = __builtin_amdgcn_mfma_i32_32x32x32_i8(g.x[ks], w.w[ks], acc, 0, 0, 0);
    if (any) {
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) {
        const v4u wu = __builtin_bit_cast(v4u, w.w[ks]) ^ 0x80808080u;
#pragma unroll
        for (int t = 0; t < 2; ++t) accf = __builtin_amdgcn_mfma_f32_32x32x16_f16(g.xf[2 * ks + t], codes_to_half8(wu, t), accf, 0, 0, 0);
      }
    }
  };

  // In iteration j: request the weights of slab j + 3 (past the end the last slab again: uniform loop body); read the fragments
  // of slab j + 1; multiply slab j; make slab j + 2 in the buffer that slab j - 2 used (a ring of four, so that every index is
  // static in a loop unrolled four times); barrier.
  Frags fr[2];
  make_slab(0, 0);
  make_slab(min(1, last), 1);
  __syncthreads();
  // the flags of the next 64 slabs as one scalar mask (bit i: slab base + i, the last slab repeated past the end)
  uint64_t any_mask = __builtin_amdgcn_ballot_w64(s_any[min(lane, last)] != 0);
  bool any_next = any_mask & 1u;
  read_frags(0, any_next, fr[0]);
  auto iteration = [&](int j, auto u_tag) {
    constexpr int u = decltype(u_tag)::value;                         // j % 4
    const bool any_cur = any_next;
    if constexpr (u == 3) {                                           // 64 is a multiple of four: only here can j + 1 start a window
      if (((j + 1) & 63) == 0) any_mask = __builtin_amdgcn_ballot_w64(s_any[min(j + 1 + lane, last)] != 0);
    }
    any_next = (any_mask >> ((j + 1) & 63)) & 1u;
    fetch_w(min(j + 3, last), f[(u + 3) & 3]);
    read_frags((u + 1) & 3, any_next, fr[(u + 1) & 1]);
    multiply(any_cur, fr[u & 1], f[u & 3]);
    make_slab(min(j + 2, last), (u + 2) & 3);
    __syncthreads();
  };
  // (whole groups of four without a way out in between: with an exit after every iteration the compiler waits for weights
  // requested one iteration earlier instead of three)
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

  // ---- outputs.  C layout of the 32x32 MFMA: lane = column n (lane % 32), register e = row 8 (e / 4) + 4 (lane / 32) + (e % 4)
  const float c = n < a.N ? a.c[n] : 0.0f;
  const float b = (!kSplit && a.bias && n < a.N) ? half_lo_to_float(a.bias[n]) : 0.0f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {                                       // (rows 8 and on are not there)
    const int m = 4 * lg + e;
    if (m < a.M && n < a.N) {
      const float y = (float)acc[e] * (s_r[m] * (c / 16129.0f)) + accf[e] * (c / 127.0f);
      if constexpr (kSplit)
        a.partial[((size_t)split * a.M + m) * a.N + n] = y;
      else
        a.Y[(size_t)m * a.ldy + n] = (uint16_t)float_to_half_bits(y + b);
      if constexpr (kTap) {
        if constexpr (kSplit)
          atomicAdd(a.tap_acc + (size_t)m * a.N + n, acc[e]);         // tap buffer zeroed by the launcher
        else
          a.tap_acc[(size_t)m * a.N + n] = acc[e];
      }
    }
  }
}

// Ranges of K: a workgroup takes 0.45 us per slab, or its share of what HBM delivers (6.2 TB/s), and the fp32 sums of a range
// cost their 8 bytes per output at 3 TB/s: the sum of both is least at sqrt(0.45 slabs / cost of a range), unless HBM is busy
// with fewer workgroups.  Counted for 32 rows, not for the rows of the call, so that a workspace sized for more rows gives
// the same ranges.
SkinnyPlan plan_skinny(int K, int N) {
  SkinnyPlan p;
  p.n_slabs = packed_k(K) / kSlabBytes;
  p.tiles_n = packed_n(N) / 256;
  const int enough = ceil_div((int)(0.45 * 6.2e6 / kBlockBytes), p.tiles_n);          // workgroups per tile that keep HBM busy
  const int cheapest = (int)(sqrt(0.45 * p.n_slabs * 3.0e6 / (32.0 * N * 8)) + 0.5);
  const int best = max(1, min(min(enough, cheapest), min(device_cu_count() / p.tiles_n, p.n_slabs / 2)));
  p.slabs_per_split = ceil_div(p.n_slabs, best);
  p.splits = ceil_div(p.n_slabs, p.slabs_per_split);
  return p;
}

// k_gemm_panel: a range per compute unit, at least eight slabs each; the columns of a range have to fit in LDS.  splits 0: not
// for this call.
SkinnyPlan plan_panel(int M, int K, int N) {
  const int Kpad = packed_k(K), cus = device_cu_count();
  SkinnyPlan p = {Kpad / kSlabBytes, packed_n(N) / 256, 0, 0};
  p.slabs_per_split = ceil_div(p.n_slabs, max(1, min(p.n_slabs / 8, cus / p.tiles_n)));
  const int splits = ceil_div(p.n_slabs, p.slabs_per_split);
  const bool fits = M >= 1 && M <= kPanelMaxM && p.slabs_per_split <= kPanelMaxSlabs && M * p.slabs_per_split <= kPanelMaxRowSlabs;
  // The rows go through every workgroup, so not with too many of them; a slab takes it longer than k_gemm_decode (five rows and
  // more, heavy-tailed), so only with short ranges or nearly every compute unit at work; and what it saves is a launch or two,
  // which large weights do not show.  us, this kernel / k_prep_rows and k_gemm_decode: 8 x 11008 -> 4096 17.5 / 19.5, 3 x 16384 ->
  // 2048 14.1 / 17.4, 5 x 512 -> 57344 10.7 / 14.5; at the lines 8 x 24576 -> 2048 (197k elements) 20.6 / 21.9, 8 x 65536 -> 1024
  // (524k) 32.3 / 28.9; 8 x 4096 -> 24576 (192 workgroups, 32 slabs) 28.2 / 25.7, 3 x 17920 -> 6656 (234, 32) 28.1 / 30.6; 4 x
  // 20480 -> 8192 (168 MB) 36.0 / 36.9, 4 x 24576 -> 8192 (201 MB) 43.3 / 40.5; two rows of 36864 -> 8192 56.9 / 60.6, of 49152 ->
  // 8192 77.8 / 75.3.
  const bool saves = (((size_t)Kpad * N <= 200000000 && M * Kpad <= 200000) || (M <= 2 && M * Kpad <= 80000)) &&
                     (p.slabs_per_split <= 16 || 10 * p.tiles_n * splits >= 9 * cus);
  if (fits && saves) p.splits = splits;
  return p;
}

template <int kBM>
static hipError_t prepare_decode() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_gemm_decode<kBM>), hipFuncAttributeMaxDynamicSharedMemorySize, DecodeCfg<kBM>::LDS_BYTES);
}
template <int kBM>
static hipError_t launch_decode(const SkinnyArgs& a, int splits, hipStream_t stream) {
  hipLaunchKernelGGL(k_gemm_decode<kBM>, dim3(a.tiles_n * splits), dim3(DecodeCfg<kBM>::kThreads), DecodeCfg<kBM>::LDS_BYTES, stream, a);
  return hipGetLastError();
}

hipError_t prepare_skinny_kernels() {
  static std::atomic<bool> attr_set[64] = {};                      // setting an attribute twice is harmless
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (attr_set[dev]) return hipSuccess;
  hipError_t e = prepare_decode<32>();
  if (e == hipSuccess) e = prepare_decode<64>();
  if (e == hipSuccess) e = prepare_decode<128>();
  if (e == hipSuccess) e = prepare_rows_kernels();
  if (e == hipSuccess) attr_set[dev] = true;
  return e;
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

// the sums of the ranges, and the rest of the layer
static hipError_t launch_finalize(const SkinnyArgs& a, int splits, hipStream_t stream) {
  if (a.codes) {
    const FinalizedHalves src = {a.partial, splits, a.N, (size_t)a.M * a.N, a.bias, a.residual, a.ldr, a.Y};
    return launch_finalize_coded(src, a.code_block, a.codes, a.code_absmax, a.flag_reset, a.Kpad, stream);
  }
  hipLaunchKernelGGL(k_skinny_finalize, dim3(ceil_div(a.N, 256), a.M), dim3(256), 0, stream, a.partial, splits,
                     a.M, a.N, a.bias, a.lora_P, a.lora_splits, a.lora_B, a.lora_r, a.lora_T_user, a.residual, a.ldr, a.gelu, a.Y, a.ldy,
                     a.flag_reset, a.Kpad);
  return hipGetLastError();
}
static void clear_tap(const SkinnyArgs& a, hipStream_t stream) {
  const size_t n = (size_t)a.M * a.N;
  if (a.tap_acc) hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, stream, a.tap_acc, n);
}

hipError_t launch_gemm_skinny(SkinnyArgs a, const SkinnyPlan& plan, hipStream_t stream) {
  a.n_slabs = plan.n_slabs;
  a.tiles_n = plan.tiles_n;
  a.slabs_per_split = plan.slabs_per_split;
  if (a.M < 1 || a.M > kSkinnyMaxM || !a.partial || !a.X) return hipErrorInvalidValue;
  if (hipError_t e = prepare_skinny_kernels(); e != hipSuccess) return e;
  clear_tap(a, stream);
  hipError_t e = a.M <= 32 ? launch_decode<32>(a, plan.splits, stream) : a.M <= 64 ? launch_decode<64>(a, plan.splits, stream) : launch_decode<128>(a, plan.splits, stream);
  // the sums go through memory whether K is split or not: the kernel that adds them is the rest of the layer (and it puts the
  // column flags back to zero, which every workgroup of the kernel before it reads)
  return e == hipSuccess ? launch_finalize(a, plan.splits, stream) : e;
}

hipError_t launch_gemm_panel(SkinnyArgs a, const SkinnyPlan& plan, hipStream_t stream) {
  a.n_slabs = plan.n_slabs;
  a.tiles_n = plan.tiles_n;
  a.slabs_per_split = plan.slabs_per_split;
  if (plan.splits < 1 || a.M < 1 || a.M > kPanelMaxM || !a.partial || !a.X || plan.slabs_per_split > kPanelMaxSlabs ||
      a.M * plan.slabs_per_split > kPanelMaxRowSlabs)
    return hipErrorInvalidValue;
  const bool sums = plan.splits > 1 || a.lora_r > 0 || a.residual || a.codes || a.gelu;
  const dim3 grid(plan.tiles_n * plan.splits), block(kPanelThreads);
  if (sums) {
    clear_tap(a, stream);
    if (a.tap_acc) hipLaunchKernelGGL((k_gemm_panel<true, true>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((k_gemm_panel<true, false>), grid, block, 0, stream, a);
  } else {
    if (a.tap_acc) hipLaunchKernelGGL((k_gemm_panel<false, true>), grid, block, 0, stream, a);
    else hipLaunchKernelGGL((k_gemm_panel<false, false>), grid, block, 0, stream, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !sums) return e;
  a.flag_reset = nullptr;                                             // (done by the kernel before, which does not read them)
  return launch_finalize(a, plan.splits, stream);
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
constexpr int kRowsCodePad = 64, kRowsHalfPad = 72;   // bytes, halves (multiples of 16 bytes)
template <int kM, int kChunks>
__global__ __launch_bounds__(kRowsWaves * kWave) void k_gemm_rows(const SkinnyArgs a) {
  constexpr int WAVES = kRowsWaves, kThreads = WAVES * kWave, kAhead = 3;
  extern __shared__ __attribute__((aligned(16))) int8_t s_ops[];     // rows_lds_bytes: operands, chunk flags, sums
  __shared__ uint8_t s_any[MMD8_MAX_K / kSlabBytes];
  __shared__ uint32_t s_part[kM][WAVES];
  __shared__ float s_r[kM], s_scale[kM];
  __shared__ __attribute__((aligned(16))) uint16_t s_T[kM][kLoraMaxRank];
  static_assert(kM * kLoraMaxRank <= kRowsWaves * kWave, "a thread per value of T");
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // the operand row / output column a lane stands for, and which 16-byte piece of the slab it holds
  const int lr = lane & 15, lg = lane >> 4;
  const int n_slabs = a.n_slabs, Kpad = n_slabs * kSlabBytes;
  const int M = kM == 1 ? 1 : a.M;
  reset_column_flags(a.flag_reset, Kpad);
  const int row_chunks = Kpad / 8, all_chunks = M * row_chunks;
  // (rows a little further apart than they are long: a fragment read takes the same piece of every row, and rows whose
  // distance is a multiple of 256 bytes keep it in the same banks: 57 % of the LDS cycles at eight rows, 4096 -> 4096 14.2 us,
  // 11.7 now)
  const int code_row = Kpad + kRowsCodePad, xf_row = Kpad + kRowsHalfPad;
  int8_t* s_code = s_ops;                                            // [M][code_row]
  uint16_t* s_xf = reinterpret_cast<uint16_t*>(s_ops + (size_t)M * code_row);    // [M][xf_row]
  uint8_t* s_over = reinterpret_cast<uint8_t*>(s_xf + (size_t)M * xf_row);     // [all_chunks]: bits "at or above the threshold" (kM > 1)
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
    uint32_t bits = 0;                                                // element j in the low half: bit j, in the high half: bit 15 + j
#pragma unroll
    for (int w = 0; w < 4; ++w) {   // per half, wraps mod 2^16: entries below the threshold get the top bit
      raw[i][w] = ok ? raw[i][w] : 0u;
      const us2 d = (us2)(__builtin_bit_cast(us2, raw[i][w] & 0x7fff7fffu) - th2);
      t = __builtin_elementwise_max(t, d);
      const uint32_t below = __builtin_bit_cast(uint32_t, (ss2)(__builtin_bit_cast(ss2, d) >> 15));   // 0xffff per such entry
      bits |= ~below & (0x00020001u << (2 * w));
    }
    over[i] = ok ? (bits | bits >> 16) & 0xffu : 0u;
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
      uint32_t code[2], xf[4], mask[2];                                // mask: 0xff per critical column
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const uint32_t ones = (((crit >> (4 * q)) & 0xfu) * 0x00204081u) & 0x01010101u;   // bit j to byte j
        mask[q] = (ones << 8) - ones;
        // (an entry of a column that is not critical is at most the row's largest)
        code[q] = to_code_word(raw[i][2 * q], raw[i][2 * q + 1], sc) & ~mask[q];
#pragma unroll
        for (int w = 0; w < 2; ++w)
          xf[2 * q + w] = raw[i][2 * q + w] & __builtin_amdgcn_perm(0u, mask[q], w ? 0x03030202u : 0x01010000u);
      }
      *reinterpret_cast<v2u*>(s_code + (size_t)m * code_row + k) = v2u{code[0], code[1]};
      *reinterpret_cast<v4u*>(s_xf + (size_t)m * xf_row + k) = v4u{xf[0], xf[1], xf[2], xf[3]};
      if (crit) s_any[k >> 6] = 1;
    }
  }
  __syncthreads();

  // ---- the products
  v4i acc = v4i{0, 0, 0, 0};
  v4f accf = v4f{0.0f, 0.0f, 0.0f, 0.0f};
  const bool row_live = lr < M;
  const int row = row_live ? lr : 0;                                  // lanes beyond M read row 0 and feed zeros
  const int8_t* my_code = s_code + (size_t)row * code_row + lg * 16;
  const uint16_t* my_xf = s_xf + (size_t)row * xf_row + lg * 16;
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
  if ((int)threadIdx.x < M * a.lora_r) {                              // an adapter's T
    const int m = (int)threadIdx.x / a.lora_r, j = (int)threadIdx.x % a.lora_r;
    const uint32_t t = sum_low_rank_activation(a.lora_P, a.lora_splits, M, m, j);
    s_T[m][j] = (uint16_t)t;
    if (a.lora_T_user && blockIdx.x == 0) a.lora_T_user[threadIdx.x] = (uint16_t)t;
  }
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
        const v4u t = *reinterpret_cast<const v4u*>(&s_T[out_m][j]);
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
  return (size_t)M * (3 * Kpad + kRowsCodePad + 2 * kRowsHalfPad) + (M > 1 ? round_up(M * Kpad / 8, 16) : 0) + (size_t)tiles * 2 * kRowsWaves * M * 16 * 4;
}
// most tiles a workgroup can have: their sums in LDS, an output per thread
static int rows_tiles_max(int M, int Kpad) {
  const long room = (long)kRowsMaxLds - (long)rows_lds_bytes(M, Kpad, 0);
  return room <= 0 ? 0 : (int)min(room / (2 * kRowsWaves * M * 16 * 4), (long)(kRowsWaves * kWave / (16 * M)));
}
// Where a compute unit holds the sums of all its tiles, so that it prepares once; a single row wherever it fits (8192 -> 57344 at
// four rows, where it would prepare twice, 93 us, with K split 80; 24576 -> 8192 at two rows 44.1 and 41.4; a 7B layer of six rows
// 65 us with every linear in this kernel, 71 split).  Left to the kernels that split K, us here / there:
//   fewer slabs than waves and many tiles: sixteen sums per tile, most of them zeros.  512 -> 57344 at three rows 11.1 / 9.9
//   (28672: 8.0 / 8.5), 96 -> 65536 at four 11.5 / 7.0;
//   long rows in a workgroup's registers, five of them and more, or few workgroups: 8192 -> 8192 at five rows 21.4 / 19.0 (6144 ->
//   8192 at six 16.7 / 17.0, 11008 -> 8192 at four 21.7 / 22.8); 24576 -> 1024 at two 16.7 / 15.5 (4096: 23.6 / 25.5).
bool rows_kernel_fits(int M, int Kpad, int N) {
  if (M < 1 || M > kRowsMaxM || M * Kpad / 8 > kRowsMaxChunks * kRowsWaves * kWave) return false;
  const int n_tiles = ceil_div(N, 16), cus = device_cu_count(), tiles = ceil_div(n_tiles, cus), n_slabs = Kpad / kSlabBytes;
  if (rows_tiles_max(M, Kpad) < (M == 1 ? 1 : tiles)) return false;
  if (M > 1 && n_slabs < kRowsWaves && 2 * tiles > 3 * n_slabs) return false;
  return M * Kpad <= 40000 || M == 4 || (M < 4 && 4 * n_tiles > cus);
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
  hipError_t e = prepare_rows_of<1, 1, 2, 3, 4, kRowsMaxChunks>();
  if (e == hipSuccess) e = prepare_rows_of<2, 1, 2, 3, 4, kRowsMaxChunks>();
  if (e == hipSuccess) e = prepare_rows_of<4, 1, 2, 3, 4, kRowsMaxChunks>();
  if (e == hipSuccess) e = prepare_rows_of<8, 1, 2, 3, 4, kRowsMaxChunks>();
  if (e == hipSuccess) attr_set[dev] = true;
  return e;
}

template <int kM>
static hipError_t launch_rows_of(const SkinnyArgs& a, int chunks, int grid, size_t lds, hipStream_t stream) {
  const dim3 g(grid), b(kRowsWaves * kWave);
  if (chunks <= 1) hipLaunchKernelGGL((k_gemm_rows<kM, 1>), g, b, lds, stream, a);
  else if (chunks <= 2) hipLaunchKernelGGL((k_gemm_rows<kM, 2>), g, b, lds, stream, a);
  else if (chunks <= 3) hipLaunchKernelGGL((k_gemm_rows<kM, 3>), g, b, lds, stream, a);
  else if (chunks <= 4) hipLaunchKernelGGL((k_gemm_rows<kM, 4>), g, b, lds, stream, a);
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
