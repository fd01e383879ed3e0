// int8 MFMA GEMM with the fused mixed-decomposition epilogue ("Compression techniques", item 2).
//
//   acc[m,n] = sum_k Xq[m,k] Wt[n,k]                      v_mfma_i32_32x32x32_i8, exact
//   Y[m,n]   = f16( acc r[m] c[n] / 127^2                  outer-product dequantization
//                   + sum_j X[m,O_j] f16(Wt[n,O_j] c[n]/127)   v_mfma_f32_32x32x16_f16 on the critical columns
//                   + bias[n] )
//
// Both operands are K-contiguous int8 codes in the blocked layout of operand_layout.h, padded to
// whole tiles, so the main loop has no bounds checks.  A workgroup owns one BM x BN tile of Y.
// K is walked in slabs of 64 bytes.  A slab of both operands goes from global memory straight
// into LDS (global_load_lds_dwordx4: no register staging, every wave instruction copies 1 KB that
// is contiguous in HBM) through a ring of LDS buffers, two to four slabs ahead of the MFMAs.  The
// blocks are fragment-major already in HBM: the 64 lanes of an MFMA operand read 64 consecutive
// 16-byte pieces.  A lane's 16 bytes feed one operand row of the 32x32x32 MFMA; the k order
// inside the instruction is irrelevant as long as both operands use the same piece for the same
// lane group, which they do.
//
// One kernel, k_gemm_mixed, instantiated for several tile configurations (256 x 256 with eight waves for
// large problems, smaller tiles for small ones); fragments are double-buffered in registers, by k-steps or, where the
// wave tile is small enough, by whole slabs.
#include <atomic>
#include <type_traits>
#include <utility>

#include "codec_device.h"
#include "common.h"
#include "gemm.h"
#include "launchers.h"
#include "operand_layout.h"
#include "skinny.h"

namespace mmd8 {

// the code table of the blockwise encoder, for outputs that leave in coded form
__device__ const DynamicCode kExitCode = make_dynamic_code();

constexpr int BK = 64;                  // bytes of K per slab
constexpr int CPR = BK / 16;            // 16-byte chunks per LDS row
constexpr int ROWS_PER_DMA = kWave / CPR;

static_assert(BK == kSlabBytes, "one LDS slab is one slab of the packed operands");

// Address of the first byte that DMA instruction j of `wave` copies for slab 0 of an operand tile
// whose first row is row0 (a multiple of 16 inside one panel): 16 rows x 64 bytes, contiguous.
__device__ __forceinline__ const int8_t* dma_source(const int8_t* base, int row0, int n_slabs, int j, int waves, int wave,
                                           int lane) {
  return base + (size_t)(row0 >> 8) * n_slabs * kBlockBytes +
         (size_t)((row0 & 255) + (j * waves + wave) * ROWS_PER_DMA) * kSlabBytes + lane * 16;
}

template <int BM_, int BN_, int WAVES_M_, int WAVES_N_, int STAGES_, int WAVES_PER_SIMD_>
struct GemmCfg {
  static constexpr int kWavesPerSimd = WAVES_PER_SIMD_;           // register budget: 512 / this
  static constexpr int BM = BM_, BN = BN_, WAVES_M = WAVES_M_, WAVES_N = WAVES_N_;
  static constexpr int kWaves = WAVES_M * WAVES_N;
  static constexpr int kThreads = kWaves * kWave;
  static constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  static constexpr int TI = WM / 32, TJ = WN / 32;                 // MFMA tiles per wave
  static constexpr int NKS = BK / 32;                              // MFMA k-steps per slab
  static constexpr int A_BYTES = BM * BK, B_BYTES = BN * BK;
  static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
  static constexpr int kStages = STAGES_;
  static constexpr int RING_BYTES = STAGE_BYTES * kStages;
  static constexpr int R_BYTES = 1024;                             // 256 row scales, one DMA instruction
  static constexpr int LDS_BYTES = RING_BYTES + R_BYTES;
  static constexpr int A_DMA = BM / ROWS_PER_DMA / kWaves;         // DMA instructions per wave per slab
  static constexpr int B_DMA = BN / ROWS_PER_DMA / kWaves;
  static constexpr int DMA_PER_SLAB = A_DMA + B_DMA;
  // Small wave tiles have registers left for the fragments of a whole slab next to those being multiplied: a slab is
  // read from LDS while the one before it is multiplied, and its buffer is free one iteration earlier.
  static constexpr bool kSlabAhead = TI * TJ <= 4;
  static constexpr int kAhead = kSlabAhead ? kStages : kStages - 1;  // slabs requested ahead of the MFMAs
  static_assert(BM % (ROWS_PER_DMA * kWaves) == 0 && BN % (ROWS_PER_DMA * kWaves) == 0, "tile/wave mismatch");
  static_assert(WM % 32 == 0 && WN % 32 == 0, "wave tile must be whole MFMA tiles");
  static_assert(NKS == 2, "fragment buffering below is written for two k-steps per slab");
  static_assert(kStages >= 3 && (kStages - 1) * DMA_PER_SLAB <= 63, "the requests in flight fit the wait instruction's count");
  static_assert(LDS_BYTES <= 160 * 1024, "LDS");
  static_assert(BM <= 256, "row scales are staged with one 1 KB request");
  // gather staging of critical columns beyond the slab: [rows][16 k] fp16 for both operands
  static_assert((BM + BN) * 32 <= RING_BYTES, "epilogue staging must fit in the slab buffers");
};

// The tile configurations, by the number a caller can force one with (gemm.h).  Eight waves each, two to a SIMD, one of which
// multiplies while the other waits: 128 x 128 tiles of four waves (64 x 64 each, one to a SIMD, a three-slab ring) took 37.2 us
// instead of 32.6 for 256 x 4096 x 12288, 37.7 instead of 32.3 for 512 x 4096 x 6144, 26.5 instead of 22.6 for 128 x 4096 x 4096 with
// original weight rows; with heavy-tailed rows 40.7 instead of 35 for 256 x 2816 x 2048 and 63.3 instead of 59.6 for 256 x
// 4096 x 12288.  (Held to 128 registers, two workgroups to a compute unit, the walk spills: 69.7 for the last of these.)
using Cfg0 = GemmCfg<128, 128, 2, 4, 4, 2>;
using Cfg1 = GemmCfg<256, 128, 4, 2, 3, 2>;
using Cfg2 = GemmCfg<128, 256, 2, 4, 3, 2>;
using Cfg3 = GemmCfg<256, 256, 2, 4, 3, 2>;
using Cfg4 = GemmCfg<256, 256, 2, 4, 4, 2>;   // the large tile: whole rounds of one tile per CU
using Cfg5 = GemmCfg<128, 256, 2, 4, 4, 2>;   // remainders and less than one round of large tiles

// own requests older than the newest kVm have landed, own LDS reads have returned; after the
// barrier that holds for every wave of the workgroup
template <int kVm>
__device__ inline void wait_slab_and_sync() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" : : "n"(kVm) : "memory");
}

// Tile assignment.  Consecutive workgroup ids land on different XCDs (8 of them, each with its own L2), so XCD x
// gets the ids x, x + 8, ...: a contiguous run of the tile order below, 32 tiles (one per CU) at a time.  The order
// walks blocks of 8 tile rows x 4 tile columns (bands of 4 columns; inside a band blocks of 8 rows; inside a
// block rows fastest), so the 32 tiles an XCD works on at once share 8 activation panels and 4 weight panels:
// 12 panel streams through its L2 instead of the 18 of a plain rows-fastest order with 16 tile rows (measured on
// the 70B-shaped linears at 4096 tokens: 1.4-2.1 % faster; identical for up to 8 tile rows).
// Split K: the ranges of K one after the other, each over all tiles, so that an XCD reads few ranges of both operands
// and a weight byte mostly comes into one L2 only.
__device__ inline bool tile_of_block(const GemmArgs& a, int bid, int& tm, int& tn, int& split) {
  constexpr int kBlockRows = 8, kBandCols = 4;
  const int n_tiles = a.tiles_m * a.tiles_n;
  const int per_xcd = ceil_div(n_tiles * a.splits, 8);
  int logical = (bid % 8) * per_xcd + bid / 8;
  if (logical >= n_tiles * a.splits) return false;
  split = logical / n_tiles;
  logical -= split * n_tiles;
  const int band_tiles = a.tiles_m * kBandCols;                    // (every band but the last is full)
  const int band = logical / band_tiles;
  const int w = min(kBandCols, a.tiles_n - band * kBandCols);      // width of this band
  const int q = logical - band * band_tiles;                       // index inside the band
  const int full_blocks = a.tiles_m / kBlockRows, rest_rows = a.tiles_m - full_blocks * kBlockRows;
  if (q < full_blocks * kBlockRows * w) {
    const int r = q % (kBlockRows * w);
    tm = (q / (kBlockRows * w)) * kBlockRows + r % kBlockRows;
    tn = band * kBandCols + r / kBlockRows;
  } else {                                                         // the last, shorter block of rows
    const int r = q - full_blocks * kBlockRows * w;
    tm = full_blocks * kBlockRows + r % rest_rows;
    tn = band * kBandCols + r / rest_rows;
  }
  return true;
}

// ------------------------------------------------------------------------------------------------
// Epilogue pieces.  C layout of the 32x32 MFMA: a lane holds column (lane % 32); register e holds
// row 8 (e / 4) + 4 (lane / 32) + (e % 4).  The accumulators stay where the MFMAs left them: they
// are dequantized in place (the registers then hold fp32 bits), the fp16 MFMAs of the critical
// columns accumulate onto them in place, and each 32x32 tile is converted and stored on its own.
// ------------------------------------------------------------------------------------------------
template <class Cfg>
struct WavePos {
  int m0, n0, wm, wn, lane, lr, lg, mw, nw;
  __device__ WavePos(int m0_, int n0_, int wave, int lane_)
      : m0(m0_), n0(n0_), wm(wave / Cfg::WAVES_N), wn(wave % Cfg::WAVES_N), lane(lane_), lr(lane_ & 31),
        lg(lane_ >> 5), mw(m0_ + (wave / Cfg::WAVES_N) * Cfg::WM), nw(n0_ + (wave % Cfg::WAVES_N) * Cfg::WN) {}
};

// (split K: the ranges add up in a buffer that the launcher zeroed; integers, so in any order)
template <class Cfg, bool kSplit>
__device__ __forceinline__ void tap_accumulators(const GemmArgs& a, const WavePos<Cfg>& p, v16i (&acc)[Cfg::TI][Cfg::TJ]) {
#pragma unroll
  for (int i = 0; i < Cfg::TI; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::TJ; ++j) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int m = p.mw + i * 32 + 8 * (e / 4) + 4 * p.lg + (e % 4), n = p.nw + j * 32 + p.lr;
        if (m < a.M && n < a.N) {
          if constexpr (kSplit)
            atomicAdd(a.tap_acc + (size_t)m * a.tap_ld + n, acc[i][j][e]);
          else
            a.tap_acc[(size_t)m * a.tap_ld + n] = acc[i][j][e];
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
}

// acc := bits( acc * r[m] * (c[n] / 127^2) ).  r_tile points at the 256 (or fewer) row scales of
// this workgroup tile, in LDS or in global memory.
template <class Cfg, class RPtr>
__device__ __forceinline__ void dequantize_in_place(const WavePos<Cfg>& p, v16i (&acc)[Cfg::TI][Cfg::TJ], RPtr r_tile,
                                           const float (&cs)[Cfg::TJ]) {
#pragma unroll
  for (int i = 0; i < Cfg::TI; ++i) {
    float rm[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const v4f v = *reinterpret_cast<const v4f*>(r_tile + p.wm * Cfg::WM + i * 32 + 8 * q + 4 * p.lg);
      rm[4 * q] = v[0], rm[4 * q + 1] = v[1], rm[4 * q + 2] = v[2], rm[4 * q + 3] = v[3];
    }
#pragma unroll
    for (int j = 0; j < Cfg::TJ; ++j) {
      v16f y;
#pragma unroll
      for (int e = 0; e < 16; ++e) y[e] = (float)acc[i][j][e] * (rm[e] * cs[j]);
      acc[i][j] = __builtin_bit_cast(v16i, y);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Critical columns j_begin .. n_out-1, 16 at a time: every thread helps to stage X[m, O_j] (fp16)
// and f16(Wt[n, O_j] c[n] / 127) for the whole tile in LDS as [row][16] fp16, then one 32x32x16
// fp16 MFMA per output tile.  General (any number of columns); the slab buffers must be free.
// A thread owns one of the 16 columns and every (kThreads / 16)-th row; all its gathers of a step are
// issued together (clamped addresses, results masked), so a step costs a few memory latencies, not one
// per element.
template <class Cfg>
__device__ __forceinline__ void gather_outlier_columns(const GemmArgs& a, const WavePos<Cfg>& p, v16i (&acc)[Cfg::TI][Cfg::TJ],
                                              int8_t* smem, int j_begin, int n_out) {
  constexpr int TI = Cfg::TI, TJ = Cfg::TJ, TILE_M = Cfg::BM, TILE_N = Cfg::BN;
  constexpr int RSTEP = Cfg::kThreads / 16;                        // rows between a thread's items
  constexpr int NX = TILE_M / RSTEP, NW = TILE_N / RSTEP;          // its rows of X, then of Wt
  static_assert(TILE_M % RSTEP == 0 && TILE_N % RSTEP == 0, "whole rows per thread");
  uint16_t* sXo = reinterpret_cast<uint16_t*>(smem);             // [TILE_M][16], then [TILE_N][16]
  uint16_t* sWo = sXo + TILE_M * 16;
  const int kk = threadIdx.x & 15, r0 = threadIdx.x >> 4;
  const int n_slabs = a.Kpad / BK;
  __syncthreads();                                               // every wave is done with the slab ring
  // (the column index of a step is asked for one step ahead, and a step's loads of X and of the weights go out
  // together: one memory latency per step instead of three)
  int k_next = j_begin + kk < n_out ? a.idx[j_begin + kk] : 0;
  for (int j0 = j_begin; j0 < n_out; j0 += 16) {
    const bool col_ok = j0 + kk < n_out;
    const int k = k_next;
    k_next = j0 + 16 + kk < n_out ? a.idx[j0 + 16 + kk] : 0;
    // eight rows at a time: enough loads in flight, few registers next to the accumulators
    constexpr int BX = NX < 8 ? NX : 8, BW = NW < 8 ? NW : 8;
    static_assert(NX % BX == 0 && NW % BW == 0, "whole batches");
    constexpr int kBatches = NX / BX > NW / BW ? NX / BX : NW / BW;
    const uint16_t* xcol = a.X + k;
    const int xld = a.ldx;
#pragma unroll 1
    for (int b = 0; b < kBatches; ++b) {
      const bool has_x = b < NX / BX, has_w = b < NW / BW;
      uint16_t xv[BX], wv[BW];
      int8_t wq[BW];
      float wc[BW];
      if (has_x) {
#pragma unroll
        for (int i = 0; i < BX; ++i) xv[i] = xcol[(size_t)min(p.m0 + r0 + (b * BX + i) * RSTEP, a.M - 1) * xld];
      }
      if (has_w) {
        if (a.W_master) {                                     // the original 16-bit rows, as they are
#pragma unroll
          for (int i = 0; i < BW; ++i)
            wv[i] = a.W_master[(size_t)k * a.ldw_master + min(p.n0 + r0 + (b * BW + i) * RSTEP, a.N - 1)];
        } else {
#pragma unroll
          for (int i = 0; i < BW; ++i) {
            const int n = min(p.n0 + r0 + (b * BW + i) * RSTEP, a.N - 1);
            wq[i] = a.Wt[packed_offset(n, k, n_slabs)];
            wc[i] = a.c[n];
          }
        }
      }
      if (has_x) {
#pragma unroll
        for (int i = 0; i < BX; ++i) {
          const int row = r0 + (b * BX + i) * RSTEP;
          sXo[row * 16 + kk] = (col_ok && p.m0 + row < a.M) ? xv[i] : (uint16_t)0;
        }
      }
      if (has_w) {
#pragma unroll
        for (int i = 0; i < BW; ++i) {
          const int row = r0 + (b * BW + i) * RSTEP;
          const uint16_t v = a.W_master ? wv[i] : (uint16_t)rounded_float_to_half_bits((float)wq[i] * (wc[i] / 127.0f));
          sWo[row * 16 + kk] = (col_ok && p.n0 + row < a.N) ? v : (uint16_t)0;
        }
      }
    }
    __syncthreads();
    v8h fxa[TI], fxb[TJ];
#pragma unroll
    for (int i = 0; i < TI; ++i)
      fxa[i] = *reinterpret_cast<const v8h*>(sXo + (p.wm * Cfg::WM + i * 32 + p.lr) * 16 + p.lg * 8);
#pragma unroll
    for (int j = 0; j < TJ; ++j)
      fxb[j] = *reinterpret_cast<const v8h*>(sWo + (p.wn * Cfg::WN + j * 32 + p.lr) * 16 + p.lg * 8);
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
        acc[i][j] = __builtin_bit_cast(
            v16i, __builtin_amdgcn_mfma_f32_32x32x16_f16(fxa[i], fxb[j], __builtin_bit_cast(v16f, acc[i][j]), 0, 0, 0));
    __syncthreads();
  }
}

// bias, rounding to fp16, and stores, through LDS (the slab buffers are free by now).  Neighbouring lanes hold
// neighbouring columns of the same rows; an even/odd lane pair swaps halves so that each lane has two adjacent
// columns (4 bytes): the even lane of row e, the odd lane of row e + 1.  A wave parks 64 (or 32) rows of its
// sub-tile at a time as fp16 rows in a region of its own and writes them out 16 bytes per lane, eight lanes
// per 128-byte row segment: a store instruction covers whole lines.  (Storing the 4-byte pairs directly
// takes four times as many store instructions and writes half lines that do not always meet in L2 before
// write-back: 2-5 % slower on the 256 x 256 tiles, 1.3 times the output in HBM write traffic.)  On the 128 x 128 tiles, whose waves
// own 32 columns, four lanes write 64 bytes of a row and another wave the rest of the line; these halves do meet: 1024 x 1024 x 4096
// writes 8.39 MB, 256 x 4096 x 12288 6.30, the output once, as with every other tile.
template <class Cfg, bool kFull>
__device__ __forceinline__ void store_tile(const GemmArgs& a, const WavePos<Cfg>& p, v16i (&acc)[Cfg::TI][Cfg::TJ],
                                      const float (&bn)[Cfg::TJ], int8_t* smem, int wave) {
  constexpr int TI = Cfg::TI, TJ = Cfg::TJ;
  constexpr int STRIDE = Cfg::WN * 2 + 16;                          // bytes per parked row (16 more: bank spread, 16-byte aligned)
  constexpr int IP = (TI >= 2 && Cfg::kWaves * 64 * STRIDE <= Cfg::RING_BYTES) ? 2 : 1;   // 32-row tiles per pass
  constexpr int RP = 32 * IP;                                       // rows per pass
  constexpr int CH = Cfg::WN / 8;                                   // 16-byte chunks per row
  static_assert(Cfg::kWaves * RP * STRIDE <= Cfg::RING_BYTES, "output staging must fit in the slab buffers");
  static_assert((RP * CH) % kWave == 0, "whole store instructions");
  int8_t* base = smem + wave * (RP * STRIDE);
  const int odd = p.lane & 1;
  __syncthreads();                                                  // every wave is done with the slab buffers
#pragma unroll
  for (int i0 = 0; i0 < TI; i0 += IP) {
#pragma unroll
    for (int ii = 0; ii < IP; ++ii) {
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const v16f y = __builtin_bit_cast(v16f, acc[i0 + ii][j]);
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const uint32_t h = float_to_half_bits(y[e] + bn[j]) | (float_to_half_bits(y[e + 1] + bn[j]) << 16);
          const uint32_t q = (uint32_t)__builtin_amdgcn_mov_dpp((int)h, 0xb1, 0xf, 0xf, true);   // quad_perm [1,0,3,2]
          const uint32_t out = odd ? ((q >> 16) | (h & 0xffff0000u)) : ((h & 0xffffu) | (q << 16));
          const int row = ii * 32 + 8 * (e / 4) + (e % 4) + 4 * p.lg + odd;
          *reinterpret_cast<uint32_t*>(base + row * STRIDE + (j * 32 + (p.lr & ~1)) * 2) = out;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int it = 0; it < RP * CH / kWave; ++it) {
      const int idx = it * kWave + p.lane, row = idx / CH, ch = idx % CH;
      const v4u v = *reinterpret_cast<const v4u*>(base + row * STRIDE + ch * 16);
      const int gm = p.mw + i0 * 32 + row, gn = p.nw + ch * 8;
      bool ok = true;
      if constexpr (!kFull) ok = gm < a.M && gn < a.N;
      if (ok) *reinterpret_cast<v4u*>(a.Y + (size_t)gm * a.ldy + gn) = v;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
}

// The same with more behind the layer: an activation (GELU, applied to the rounded output before it is parked), a
// residual, and / or an output that leaves in coded form ("Compression techniques", item 1 applied to the result
// of item 2): H = f16(Y + residual) (or Y), written where wanted, and its blockwise 8-bit codes.  Rows are parked
// as in store_tile.  Phase A (each wave on its own rows): add the residual in place, store H.  After a barrier,
// phase B: a lane takes 16 neighbouring columns of one row of the workgroup tile, whichever wave parked them,
// so that the lanes of a block are neighbours (4, 8 or 16 of them: the block maximum is a few DPP steps) and a
// wave instruction writes whole 256-byte (128-byte) rows of codes.
template <class Cfg, bool kFull>
__device__ __forceinline__ void store_tile_coded(const GemmArgs& a, const WavePos<Cfg>& p, v16i (&acc)[Cfg::TI][Cfg::TJ],
                                        const float (&bn)[Cfg::TJ], int8_t* smem, int wave) {
  constexpr int TI = Cfg::TI, TJ = Cfg::TJ;
  constexpr int STRIDE = Cfg::WN * 2 + 16;
  constexpr int CELL_BYTES = DynamicCode::kCells * 8;
  constexpr int IP = (TI >= 2 && Cfg::kWaves * 64 * STRIDE + CELL_BYTES <= Cfg::RING_BYTES) ? 2 : 1;
  constexpr int RP = 32 * IP;
  constexpr int CH = Cfg::WN / 8;
  constexpr int PARK_BYTES = Cfg::kWaves * RP * STRIDE;
  static_assert(PARK_BYTES + CELL_BYTES <= Cfg::RING_BYTES, "output staging and the code table must fit in the slab buffers");
  static_assert((RP * CH) % kWave == 0, "whole store instructions");
  constexpr int LPR = Cfg::BN / 16;                                  // lanes per row of the workgroup tile in phase B
  constexpr int TASKS = Cfg::WAVES_M * RP * LPR;
  static_assert(TASKS % Cfg::kThreads == 0 && (LPR == 8 || LPR == 16), "phase B covers the parked rows in whole rounds");
  int8_t* base = smem + wave * (RP * STRIDE);
  v2u* s_cells = reinterpret_cast<v2u*>(smem + PARK_BYTES);
  const int odd = p.lane & 1;
  const int lb = a.code_log_block;
  __syncthreads();                                                  // every wave is done with the slab buffers
  if (a.codes) stage_code_cells(s_cells, kExitCode, threadIdx.x, Cfg::kThreads);
  const uint32_t cells_biased = biased_cell_base(s_cells);
#pragma unroll
  for (int i0 = 0; i0 < TI; i0 += IP) {
#pragma unroll
    for (int ii = 0; ii < IP; ++ii) {
#pragma unroll
      for (int j = 0; j < TJ; ++j) {
        const v16f y = __builtin_bit_cast(v16f, acc[i0 + ii][j]);
#pragma unroll
        for (int e = 0; e < 16; e += 2) {
          const uint32_t h = float_to_half_bits(y[e] + bn[j]) | (float_to_half_bits(y[e + 1] + bn[j]) << 16);
          const uint32_t q = (uint32_t)__builtin_amdgcn_mov_dpp((int)h, 0xb1, 0xf, 0xf, true);   // quad_perm [1,0,3,2]
          const uint32_t out = odd ? ((q >> 16) | (h & 0xffff0000u)) : ((h & 0xffffu) | (q << 16));
          const int row = ii * 32 + 8 * (e / 4) + (e % 4) + 4 * p.lg + odd;
          *reinterpret_cast<uint32_t*>(base + row * STRIDE + (j * 32 + (p.lr & ~1)) * 2) = out;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    // The activation, on the rounded layer output: a loop of its own over the parked rows, not unrolled.  This code runs once
    // per tile and comes from memory; with the activation written out at each of a lane's elements and stepped over where
    // there is none, every element cost the fetch of its instructions (ViT-L block of 1576 rows 121 -> 116.4 us, with the
    // residual as below; no change where tiles are long: 70B-shaped layer of 4096 rows).
    if (a.gelu) {
#pragma unroll 1
      for (int it = 0; it < RP * CH / kWave; ++it) {
        const int idx = it * kWave + p.lane;
        v4u* cell = reinterpret_cast<v4u*>(base + idx / CH * STRIDE + idx % CH * 16);
        v4u v = *cell;
#pragma unroll
        for (int w = 0; w < 4; ++w) v[w] = gelu_half_pair(v[w]);
        *cell = v;
      }
    }
    // ---- phase A.  The residual is asked for four pieces at a time: between the stores of H (which may be the same array)
    // the loads would wait for each other, a memory latency each.
    if (a.residual || a.Y) {
      constexpr int kSteps = RP * CH / kWave, kBatch = kSteps < 4 ? kSteps : 4;
      static_assert(kSteps % kBatch == 0, "whole batches");
#pragma unroll
      for (int it0 = 0; it0 < kSteps; it0 += kBatch) {
        v4u res[kBatch];
        if (a.residual) {
#pragma unroll
          for (int it = 0; it < kBatch; ++it) {
            const int idx = (it0 + it) * kWave + p.lane, gm = p.mw + i0 * 32 + idx / CH, gn = p.nw + idx % CH * 8;
            const bool ok = kFull || (gm < a.M && gn < a.N);
            res[it] = *reinterpret_cast<const v4u*>(a.residual + (ok ? (size_t)gm * a.ldr + gn : (size_t)0));
          }
        }
#pragma unroll
        for (int it = 0; it < kBatch; ++it) {
          const int idx = (it0 + it) * kWave + p.lane, row = idx / CH, ch = idx % CH;
          int8_t* cell = base + row * STRIDE + ch * 16;
          v4u v = *reinterpret_cast<const v4u*>(cell);
          const int gm = p.mw + i0 * 32 + row, gn = p.nw + ch * 8;
          bool ok = true;
          if constexpr (!kFull) ok = gm < a.M && gn < a.N;
          if (a.residual) {
#pragma unroll
            for (int w = 0; w < 4; ++w)
              v[w] = float_to_half_bits(half_lo_to_float(v[w]) + half_lo_to_float(res[it][w])) |
                     (float_to_half_bits(half_hi_to_float(v[w]) + half_hi_to_float(res[it][w])) << 16);
            if (a.codes) *reinterpret_cast<v4u*>(cell) = v;
          }
          if (a.Y && ok) *reinterpret_cast<v4u*>(a.Y + (size_t)gm * a.ldy + gn) = v;
        }
      }
    }
    __syncthreads();                                                // the parked rows of every wave are final
    // ---- phase B
    if (a.codes) {
#pragma unroll
      for (int q = 0; q < TASKS / Cfg::kThreads; ++q) {
        const int t = q * Cfg::kThreads + threadIdx.x;
        const int col = (t % LPR) * 16, rowp = t / LPR, wm2 = rowp / RP, row = rowp % RP;
        const int8_t* src = smem + (wm2 * Cfg::WAVES_N + col / Cfg::WN) * (RP * STRIDE) + row * STRIDE + (col % Cfg::WN) * 2;
        const v4u h0 = *reinterpret_cast<const v4u*>(src), h1 = *reinterpret_cast<const v4u*>(src + 16);
        uint32_t m = max(chunk_absmax_pattern(h0), chunk_absmax_pattern(h1));
        m = dpp_max<0xB1>(m);                                       // 2 lanes
        m = dpp_max<0x4E>(m);                                       // 4 lanes: 64 elements
        if (lb >= 7) m = dpp_max<0x141>(m);                         // 8 lanes
        if (lb >= 8) m = dpp_max<0x140>(m);                         // 16 lanes
        const int gm = p.m0 + wm2 * Cfg::WM + i0 * 32 + row, gn = p.n0 + col;
        bool ok = true;
        if constexpr (!kFull) ok = gm < a.M && gn < a.N;
        const float am = half_lo_to_float(m);
        const float inv = (am == 0.0f) ? 0.0f : 1.0f / am;          // IEEE division
        if (ok) {
          const size_t e = (size_t)gm * a.code_ld + gn;
          if ((gn & ((1 << lb) - 1)) == 0) a.code_absmax[e >> lb] = am;
          const v2u c0 = encode_chunk(h0, inv, cells_biased), c1 = encode_chunk(h1, inv, cells_biased);
          *reinterpret_cast<v4u*>(a.codes + e) = v4u{c0[0], c0[1], c1[0], c1[1]};
        }
      }
    }
    __syncthreads();                                                // the next pass parks over these rows
  }
}

// Split K: the fp32 sums of this workgroup's range, [split][M][N]; the kernel that adds the ranges up
// (launch_add_splits) does what the stores above do.  32 lanes write 128 contiguous bytes of a row.
template <class Cfg>
__device__ __forceinline__ void store_partial(const GemmArgs& a, const WavePos<Cfg>& p, v16i (&acc)[Cfg::TI][Cfg::TJ], int split) {
#pragma unroll
  for (int i = 0; i < Cfg::TI; ++i)
#pragma unroll
    for (int j = 0; j < Cfg::TJ; ++j) {
      const v16f y = __builtin_bit_cast(v16f, acc[i][j]);
      const int n = p.nw + j * 32 + p.lr;
      float* dst = a.partial + ((size_t)split * a.M + p.mw + i * 32 + 4 * p.lg) * a.N + n;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int row = 8 * (e / 4) + (e % 4);
        if (p.mw + i * 32 + 4 * p.lg + row < a.M && n < a.N) dst[(size_t)row * a.N] = y[e];
      }
      __builtin_amdgcn_sched_barrier(0);
    }
}

// The scales and biases of a lane's columns: asked for by the constructor, waited for where they are first used (`use`).
template <class Cfg>
struct ColumnTerms {
  float c[Cfg::TJ];
  uint32_t b[Cfg::TJ];
  __device__ __forceinline__ ColumnTerms(const GemmArgs& a, const WavePos<Cfg>& p) {
#pragma unroll
    for (int j = 0; j < Cfg::TJ; ++j) c[j] = a.c[min(p.nw + j * 32 + p.lr, a.N - 1)];
#pragma unroll
    for (int j = 0; j < Cfg::TJ; ++j) b[j] = a.bias ? a.bias[min(p.nw + j * 32 + p.lr, a.N - 1)] : 0u;
  }
  __device__ __forceinline__ void use(float (&cs)[Cfg::TJ], float (&bn)[Cfg::TJ]) {
#pragma unroll
    for (int j = 0; j < Cfg::TJ; ++j) {
      asm volatile("" : "+v"(c[j]), "+v"(b[j]));                      // (the division and the conversion stay behind this point)
      cs[j] = c[j] / 16129.0f;
      bn[j] = half_lo_to_float(b[j]);
    }
  }
};

// The requests of a tile's slabs of codes.  Instruction j of a wave fills LDS rows [(j kWaves + wave) ROWS_PER_DMA,
// +ROWS_PER_DMA) of the operand tile: 1 KB, contiguous in HBM and in LDS.
template <class Cfg, bool kOnce>
struct CodeRequests {
  uint32_t lds;
  const int8_t* srcA[Cfg::A_DMA];
  const int8_t* srcB[Cfg::B_DMA];
  __device__ __forceinline__ CodeRequests(const GemmArgs& a, const WavePos<Cfg>& p, int wave, int first, uint32_t lds0)
      : lds(lds0 + wave * (kWave * 16)) {
    const int all_slabs = a.Kpad / BK;
#pragma unroll
    for (int j = 0; j < Cfg::A_DMA; ++j)
      srcA[j] = dma_source(a.Xq, p.m0, all_slabs, j, Cfg::kWaves, wave, p.lane) + (ptrdiff_t)first * kBlockBytes;
#pragma unroll
    for (int j = 0; j < Cfg::B_DMA; ++j)
      srcB[j] = dma_source(a.Wt, p.n0, all_slabs, j, Cfg::kWaves, wave, p.lane) + (ptrdiff_t)first * kBlockBytes;
  }
  // request d (0 .. DMA_PER_SLAB - 1) of the slab `pos` of the range: the A rows first, then the B rows
  __device__ __forceinline__ void issue(int pos, int stage, int d) const {
    const uint32_t base = lds + stage * Cfg::STAGE_BYTES;
    const ptrdiff_t off = (ptrdiff_t)pos * kBlockBytes;
    if (d < Cfg::A_DMA)
      dma16(srcA[d] + off, base + d * Cfg::kWaves * (kWave * 16));
    else if constexpr (kOnce)
      dma16_once(srcB[d - Cfg::A_DMA] + off, base + Cfg::A_BYTES + (d - Cfg::A_DMA) * Cfg::kWaves * (kWave * 16));
    else
      dma16(srcB[d - Cfg::A_DMA] + off, base + Cfg::A_BYTES + (d - Cfg::A_DMA) * Cfg::kWaves * (kWave * 16));
  }
};
// Slabs that a workgroup requests before anything else, the count of critical columns included, on which the rest of its
// way depends (gemm_tile, dense_tile).
__device__ inline int early_slabs(int n_slabs) { return n_slabs < 2 ? 1 : 2; }

// ------------------------------------------------------------------------------------------------
// One tile: the slabs of codes, then those of fp16 operands, then the epilogue.
// kFull: M and N are multiples of the tile, so no output store needs a bounds check.
// kTap: also write the raw int32 accumulators (parity checks).
// kCoded: the output goes through an activation, takes a residual and / or leaves in blockwise-coded form
// (store_tile_coded).
// kSplit: the workgroup multiplies one of a.splits ranges of K (slabs of codes and of fp16 operands alike) and leaves
// fp32 sums.
// ------------------------------------------------------------------------------------------------
template <class Cfg, bool kTap, bool kFull, bool kCoded, bool kSplit, bool kOnce>
__device__ __forceinline__ void gemm_tile(const GemmArgs& a, const WavePos<Cfg>& p, int wave, int split, int n_slabs, int n_out,
                                          const CodeRequests<Cfg, kOnce>& codes_of) {
  extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
  constexpr int TI = Cfg::TI, TJ = Cfg::TJ, NKS = Cfg::NKS, STAGES = Cfg::kStages;
  ColumnTerms<Cfg> column_terms(a, p);
  // Behind the slabs of codes, through the same ring: the fp16 slabs of the critical columns that are in use (32
  // columns each: at most crit_slabs of them in Xo / Wo, then at most g_slabs further ones in Xg / Wg; columns
  // beyond those are gathered after the loop) and those of a low-rank adapter (T on the activation side, B on the
  // weight side), which start at slab crit_slabs of Xo / Wo.
  const int crit_all = ceil_div(n_out, kOutlierSlab);
  const int crit_used = min(a.crit_slabs, crit_all);
  const int more_used = a.Xg ? min(a.g_slabs, crit_all - crit_used) : 0;
  const int all_fp16 = crit_used + more_used + (a.f_slabs - a.crit_slabs);
  const int first_fp16 = kSplit ? all_fp16 * split / a.splits : 0;     // ... and of fp16 operands
  const int total_slabs = n_slabs + (kSplit ? all_fp16 * (split + 1) / a.splits - first_fp16 : all_fp16);
  // from this tile's slabs in Xo / Wo to its further slabs in Xg / Wg: the same place in a panel, other panel sizes
  // (two allocations: the distance as a difference of addresses, not of pointers)
  const ptrdiff_t to_more_x = (ptrdiff_t)(reinterpret_cast<uintptr_t>(a.Xg) - reinterpret_cast<uintptr_t>(a.Xo)) +
                              (ptrdiff_t)(p.m0 >> 8) * (a.g_slabs - a.f_slabs) * kBlockBytes;
  const ptrdiff_t to_more_w = (ptrdiff_t)(reinterpret_cast<uintptr_t>(a.Wg) - reinterpret_cast<uintptr_t>(a.Wo)) +
                              (ptrdiff_t)(p.n0 >> 8) * (a.g_slabs - a.f_slabs) * kBlockBytes;

  // ---- the fp16 slabs' sources, as those of the codes
  const int8_t* srcXo[Cfg::A_DMA];
  const int8_t* srcWo[Cfg::B_DMA];
#pragma unroll
  for (int j = 0; j < Cfg::A_DMA; ++j) srcXo[j] = dma_source(reinterpret_cast<const int8_t*>(a.Xo), p.m0, a.f_slabs, j, Cfg::kWaves, wave, p.lane);
#pragma unroll
  for (int j = 0; j < Cfg::B_DMA; ++j) srcWo[j] = dma_source(reinterpret_cast<const int8_t*>(a.Wo), p.n0, a.f_slabs, j, Cfg::kWaves, wave, p.lane);
  // request d (0 .. DMA_PER_SLAB-1) of the slab at position `pos` of the ring's sequence: the A rows first, then the
  // B rows.  kFp16 says which kind of slab that position holds (known where the request is written down, so that
  // the loop over the codes carries no choice between the two)
  auto issue_dma = [&](int pos, int stage, int d, auto fp16_tag) {
    if constexpr (!decltype(fp16_tag)::value) return codes_of.issue(pos, stage, d);
    const uint32_t base = codes_of.lds + stage * Cfg::STAGE_BYTES;
    const int f = pos - n_slabs + first_fp16;                       // among the fp16 slabs in use
    // its place: slab f of Xo / Wo, slab f - crit_used of Xg / Wg, or an adapter's slab behind the crit_slabs of Xo / Wo
    ptrdiff_t off = (ptrdiff_t)(f < crit_used ? f : f - crit_used - more_used + a.crit_slabs) * kBlockBytes;
    if (f >= crit_used && f < crit_used + more_used)
      off = (d < Cfg::A_DMA ? to_more_x : to_more_w) + (ptrdiff_t)(f - crit_used) * kBlockBytes;
    if (d < Cfg::A_DMA)
      dma16(srcXo[d] + off, base + d * Cfg::kWaves * (kWave * 16));
    else
      dma16(srcWo[d - Cfg::A_DMA] + off, base + Cfg::A_BYTES + (d - Cfg::A_DMA) * Cfg::kWaves * (kWave * 16));
  };
  auto issue_slab = [&](int pos, int stage) {
#pragma unroll
    for (int d = 0; d < Cfg::DMA_PER_SLAB; ++d) {
      if (pos < n_slabs)
        issue_dma(pos, stage, d, std::false_type{});
      else
        issue_dma(pos, stage, d, std::true_type{});
    }
  };

  // ---- per-lane LDS read offsets: row (lane % 32) of an MFMA tile, piece (2 ks + lane / 32)
  int a_off[NKS], b_off[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) {
    // group of 32 rows: 2 KB = [k-step][lane] 16-byte pieces
    a_off[ks] = (p.wm * Cfg::WM / 32) * 2048 + ks * 1024 + p.lane * 16;
    b_off[ks] = Cfg::A_BYTES + (p.wn * Cfg::WN / 32) * 2048 + ks * 1024 + p.lane * 16;
  }
  v4i fa[2 * NKS][TI], fb[2 * NKS][TJ];                            // (kSlabAhead: two slabs; else two k-steps)
  // fragment q of a k-step, in the order in which the MFMAs need them: the first row's, the columns', the other rows'
  auto read_frag = [&](int stage, int ks, int buf, int q) __attribute__((always_inline)) {
    const int8_t* base = smem + stage * Cfg::STAGE_BYTES;
    if (q == 0 || q > TJ) {
      const int i = q == 0 ? 0 : q - TJ;
      fa[buf][i] = *reinterpret_cast<const v4i*>(base + a_off[ks] + i * 32 * BK);
    } else {
      fb[buf][q - 1] = *reinterpret_cast<const v4i*>(base + b_off[ks] + (q - 1) * 32 * BK);
    }
  };

  v16i acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0;

  // ---- software pipeline over the slab ring.  In iteration s slab s is being multiplied and
  // slab s + kAhead is requested into the buffer that held slab s - 1 (every wave finished
  // reading it before the barrier that ended iteration s - 1).  At the end of iteration s the
  // wave waits until only the requests younger than slab s + 1 are outstanding.
  // A wave issues in order, and a request that finds the memory queue full blocks the MFMAs
  // behind it, so the requests of a slab are spread evenly between the MFMAs of the iteration.
  // issue_tag: slab s + kAhead exists and is requested in this iteration (1: it is a slab of codes, 2: an fp16 slab;
  // 0: no request); kNext: slab s + 1 exists.
  constexpr int AHEAD = Cfg::kAhead;
  constexpr int MFMAS = TI * TJ;                                   // per k-step
  // request d of a slab goes out after MFMA number d SLOTS / DMA_PER_SLAB of the iteration
  constexpr int SLOTS = NKS * MFMAS, DPS_ = Cfg::DMA_PER_SLAB;
  static_assert(DPS_ >= 1 && DPS_ <= SLOTS, "request spreading");
  // requests of the iteration that are out before the wait in the last k-step (slot (NKS-1) MFMAS)
  constexpr int kBeforeWait = ((NKS - 1) * MFMAS * DPS_ + SLOTS - 1) / SLOTS;
  int stage = 0;
  // kFp16: slab s is one of the fp16 slabs (fp16 operands, fp32 accumulation onto the accumulators, which
  // were dequantized before the first of them)
  auto iteration = [&](int s, auto issue_tag, auto next_tag, auto fp16_tag) {
    constexpr int kIssueKind = decltype(issue_tag)::value;
    constexpr bool kIssue = kIssueKind != 0, kNext = decltype(next_tag)::value;
    constexpr bool kFp16 = decltype(fp16_tag)::value;
    const int stage1 = (stage + 1 == STAGES) ? 0 : stage + 1;
    const int stage_req = (stage == 0) ? STAGES - 1 : stage - 1;   // (s + kAhead) mod kStages
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int cur = ks & 1, nxt = cur ^ 1;
#pragma unroll
      for (int t = 0; t < MFMAS; ++t) {
        const int i = t / TJ, j = t % TJ;
        if constexpr (kFp16)
          acc[i][j] = __builtin_bit_cast(
              v16i, __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, fa[cur][i]),
                                                           __builtin_bit_cast(v8h, fb[cur][j]),
                                                           __builtin_bit_cast(v16f, acc[i][j]), 0, 0, 0));
        else
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
        // the first MFMA of the k-step goes out before any new LDS read, so the wait for its
        // fragments (read during the previous k-step) is already satisfied
        __builtin_amdgcn_sched_barrier(0);
        // last k-step of the slab: make slab s+1 visible, then prefetch its first fragments.
        // Still allowed in flight: slabs s+2 .. s+kAhead-1 in full and the part of slab
        // s+kAhead requested during the earlier k-steps of this iteration
        if (t == 0 && ks + 1 == NKS) wait_slab_and_sync<kIssue ? (AHEAD - 2) * Cfg::DMA_PER_SLAB + kBeforeWait : 0>();
        if (ks + 1 < NKS || kNext) {
#pragma unroll
          for (int q = t * (TI + TJ) / MFMAS; q < (t + 1) * (TI + TJ) / MFMAS; ++q)
            read_frag(ks + 1 < NKS ? stage : stage1, ks + 1 < NKS ? ks + 1 : 0, nxt, q);
        }
        __builtin_amdgcn_sched_barrier(0);
        // request d with ceil(d SLOTS / DPS) == slot, if there is one (at most one: DPS <= SLOTS)
        {
          const int slot = ks * MFMAS + t;
          const int d = slot * DPS_ / SLOTS;                             // the only candidate: d SLOTS / DPS in (slot - 1, slot]
          const bool here = d < DPS_ && (d * SLOTS + DPS_ - 1) / DPS_ == slot;
          if (kIssue && here) {
            __builtin_amdgcn_sched_barrier(0);
            issue_dma(s + AHEAD, stage_req, d, std::bool_constant<kIssueKind == 2>{});
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    stage = stage1;
  };
  // kSlabAhead: slab s has its fragments in set `par`; those of slab s + 1 are read into the other set, one read
  // between any two MFMAs.  With one k-step of four MFMAs between a read and its use, as the large tile has it with
  // eight, every k-step took the LDS latency: 4096 -> 22016 at 512 rows on 128 x 128 tiles 130 us, now 90.
  auto slab_step = [&](int s, auto par_tag, auto issue_tag, auto next_tag, auto fp16_tag) __attribute__((always_inline)) {
    constexpr int par = decltype(par_tag)::value, kIssueKind = decltype(issue_tag)::value;
    constexpr bool kIssue = kIssueKind != 0, kNext = decltype(next_tag)::value, kFp16 = decltype(fp16_tag)::value;
    const int stage1 = (stage + 1 == STAGES) ? 0 : stage + 1;
    // slab s + 1 has landed, and every wave has read slab s, whose buffer the requests of slab s + kAhead go to.  In
    // flight behind it: kAhead - 2 slabs, fewer once nothing is requested any more
    if constexpr (kIssue) {
      wait_slab_and_sync<(AHEAD - 2) * Cfg::DMA_PER_SLAB>();
    } else if constexpr (kNext) {
      const int behind = total_slabs - 2 - s;
      if (AHEAD > 3 && behind >= 2)
        wait_slab_and_sync<2 * Cfg::DMA_PER_SLAB>();
      else if (behind == 1)
        wait_slab_and_sync<Cfg::DMA_PER_SLAB>();
      else
        wait_slab_and_sync<0>();
    }
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
      for (int t = 0; t < MFMAS; ++t) {
        const int i = t / TJ, j = t % TJ, cur = par * NKS + ks;
        if constexpr (kFp16)
          acc[i][j] = __builtin_bit_cast(
              v16i, __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, fa[cur][i]), __builtin_bit_cast(v8h, fb[cur][j]),
                                                           __builtin_bit_cast(v16f, acc[i][j]), 0, 0, 0));
        else
          acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(fa[cur][i], fb[cur][j], acc[i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        const int slot = ks * MFMAS + t;
        if (kNext) {
          constexpr int kReads = NKS * (TI + TJ);
#pragma unroll
          for (int q = slot * kReads / SLOTS; q < (slot + 1) * kReads / SLOTS; ++q)
            read_frag(stage1, q / (TI + TJ), (par ^ 1) * NKS + q / (TI + TJ), q % (TI + TJ));
        }
        const int d = slot * DPS_ / SLOTS;
        if (kIssue && d < DPS_ && (d * SLOTS + DPS_ - 1) / DPS_ == slot)
          issue_dma(s + AHEAD, stage, d, std::bool_constant<kIssueKind == 2>{});
        __builtin_amdgcn_sched_barrier(0);
      }
    stage = stage1;
  };
  auto step = [&](int s, auto issue_tag, auto next_tag, auto fp16_tag) __attribute__((always_inline)) {
    if constexpr (!Cfg::kSlabAhead) {
      iteration(s, issue_tag, next_tag, fp16_tag);
    } else {
      // (one set after the other by copying: a choice between the two sets at run time costs 170 spilled registers)
      slab_step(s, std::integral_constant<int, 0>{}, issue_tag, next_tag, fp16_tag);
      if constexpr (decltype(next_tag)::value) {
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) {
#pragma unroll
          for (int i = 0; i < TI; ++i) fa[ks][i] = fa[NKS + ks][i];
#pragma unroll
          for (int j = 0; j < TJ; ++j) fb[ks][j] = fb[NKS + ks][j];
        }
      }
    }
  };
  using yes = std::true_type;
  using no = std::false_type;

  int issued = early_slabs(n_slabs);
  for (; issued < AHEAD && issued < total_slabs; ++issued) issue_slab(issued, issued);
  // slab 0 has landed once only the requests of the others are out
  [&]<int... kLater>(std::integer_sequence<int, kLater...>) __attribute__((always_inline)) {
    ((issued == kLater + 1 ? wait_slab_and_sync<kLater * Cfg::DMA_PER_SLAB>() : void()), ...);
  }(std::make_integer_sequence<int, AHEAD>{});
#pragma unroll
  for (int q = 0; q < (Cfg::kSlabAhead ? NKS : 1) * (TI + TJ); ++q) read_frag(0, q / (TI + TJ), q / (TI + TJ), q % (TI + TJ));
  int s = 0;
  using none = std::integral_constant<int, 0>;
  using codes = std::integral_constant<int, 1>;
  using halves = std::integral_constant<int, 2>;
  // nearly all of the time
  if constexpr (Cfg::kSlabAhead) {
    for (; s + AHEAD + 1 < n_slabs; s += 2) {
      slab_step(s, std::integral_constant<int, 0>{}, codes{}, yes{}, no{});
      slab_step(s + 1, std::integral_constant<int, 1>{}, codes{}, yes{}, no{});
    }
  }
  for (; s + AHEAD < n_slabs; ++s) step(s, codes{}, yes{}, no{});
  for (; s < n_slabs && s + AHEAD < total_slabs; ++s) step(s, halves{}, yes{}, no{});  // the first fp16 slabs requested
  for (; s < n_slabs && s + 1 < total_slabs; ++s) step(s, none{}, yes{}, no{});
  if (s < n_slabs) step(s++, none{}, no{}, no{});              // the last slab when nothing follows it
  if constexpr (kTap) tap_accumulators<Cfg, kSplit>(a, p, acc);
  float cs[TJ], bn[TJ];
  column_terms.use(cs, bn);
  dequantize_in_place<Cfg>(p, acc, a.r + p.m0, cs);
  for (; s + AHEAD < total_slabs; ++s) step(s, halves{}, yes{}, yes{});
  for (; s + 1 < total_slabs; ++s) step(s, none{}, yes{}, yes{});
  if (s < total_slabs) step(s, none{}, no{}, yes{});
  // What follows writes the slab buffers, and begins with a barrier: every wave has then read its last fragments.  (The
  // sums of a range go straight from registers.)  With K split the last range gathers the columns beyond the slabs.
  if (n_out > kOutlierSlab * (crit_used + more_used) && (!kSplit || split == a.splits - 1))
    gather_outlier_columns<Cfg>(a, p, acc, smem, kOutlierSlab * (crit_used + more_used), n_out);
  if constexpr (kSplit)
    store_partial<Cfg>(a, p, acc, split);
  else if constexpr (kCoded)
    store_tile_coded<Cfg, kFull>(a, p, acc, bn, smem, wave);
  else
    store_tile<Cfg, kFull>(a, p, acc, bn, smem, wave);
}

// Input with very many critical columns (heavy-tailed activations: dense_critical_path; no fp16 slab was prepared
// then).  Both products of the method in one walk over K, 64 columns (a slab) at a time:
//   int8:   the codes of X (critical columns hold zeros) times the weight codes, exact, in accumulators of its own;
//   16-bit: the rows of X itself times the same weight codes, those of columns that are not critical masked to zero (in
//           such a column every entry is below the threshold, hence finite), turned into fp16 integers in registers
//           (codes_to_half8) as the decode kernels do.  The column's step c[n] / 127
//           is applied once to the fp32 sum (against the prepared slabs the weights are not rounded to fp16 after
//           scaling: at most 2^-11 relative per term).
// A tile is 128 rows high, a wave owns 64 x 64 of it (two sets of four 32 x 32 accumulators: 128 registers; 64 x 32 where it is
// 128 columns wide), and
// everything of a slab comes through one ring of three LDS buffers by global_load_lds_dwordx4, two slabs ahead:
// codes and weight codes as in the main loop, the rows of X 128 bytes per row, eight rows per instruction.  Row R
// keeps its 16-byte piece q at place q ^ (R / 2 % 8), which the per-lane source address arranges, so that 16 lanes of a
// fragment read (neighbouring rows, the same piece) meet every bank once.  The masks of 256 slabs at a time are expanded into LDS (a
// byte per column).
// What bounds it: the 24 MFMAs of a wave and slab need 1536 cycles per SIMD (0.64 us at 2.4 GHz).
template <int kBN>
struct DenseCfg {
  using Tile = typename std::conditional<kBN == 256, Cfg5, Cfg0>::type;   // wave positions and the output stages
  static_assert(Tile::BM == 128 && Tile::BN == kBN && Tile::WM == 64 && Tile::kWaves == 8, "128 rows, eight waves of 64 rows");
  static constexpr int kCodes = 128 * BK, kRows = 128 * BK * 2, kWeights = kBN * BK;
  // a ring of codes and weight codes, laid out like that of the tile configuration (whose first slabs are requested before it
  // is known that the walk is taken), and one of rows of X behind it
  static constexpr int kStages = 3, kStage = kCodes + kWeights, kRowsAt = kStages * kStage, kMasksAt = kRowsAt + kStages * kRows;
  static_assert(kStage == Tile::STAGE_BYTES && kCodes == Tile::A_BYTES, "as in the tile's own ring");
  static constexpr int kMaskSlabs = 256;
  static constexpr int LDS_BYTES = kMasksAt + kMaskSlabs * BK;
  static constexpr int X_DMA = 128 * BK * 2 / 1024 / Tile::kWaves;
  static constexpr int kPerSlab = Tile::A_DMA + X_DMA + Tile::B_DMA;       // requests per wave and slab
  static_assert(LDS_BYTES >= Tile::kWaves * 64 * (Tile::WN * 2 + 16) + DynamicCode::kCells * 8 && LDS_BYTES <= 160 * 1024,
                "LDS (the output stages need that much of it at most)");
};

// early: early_slabs() slabs of codes have been requested into the ring.
template <int kBN, bool kOnce>
__device__ __forceinline__ void dense_tile(const GemmArgs& a, int m0, int n0, int split, int8_t* smem, bool early) {
  using D = DenseCfg<kBN>;
  using Cfg = typename D::Tile;
  constexpr int TI = Cfg::TI, TJ = Cfg::TJ;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const WavePos<Cfg> p(m0, n0, wave, lane);
  const int n_slabs = a.Kpad / BK;
  const int first = split * a.slabs_per_split, end = min(first + a.slabs_per_split, n_slabs), last = end - 1;
  int8_t* s_mask = smem + D::kMasksAt;

  const uint32_t lds0 = (uint32_t)(uintptr_t)smem + wave * (kWave * 16);
  // the codes: a scalar address per slab and a constant offset per lane and request (the loop's vector instructions
  // are what it has to save); the rows of X: a pointer per request
  const int8_t* baseA = dma_source(a.Xq, m0, n_slabs, 0, Cfg::kWaves, wave, 0);
  const int8_t* baseB = dma_source(a.Wt, n0, n_slabs, 0, Cfg::kWaves, wave, 0);
  const uint16_t* srcX[D::X_DMA];
  const int piece = 8 * ((lane & 7) ^ (4 * (wave & 1) + (lane >> 4)));   // first column of this lane's piece of a row
#pragma unroll
  for (int j = 0; j < D::X_DMA; ++j)
    srcX[j] = a.X + (size_t)min(m0 + 8 * (j * Cfg::kWaves + wave) + (lane >> 3), a.M - 1) * a.ldx + piece;
  const int whole_slabs = a.K / BK;
  // request d of slab s into buffer `stage`
  auto request = [&](int s, int stage, int d) __attribute__((always_inline)) {
    const uint32_t dst = lds0 + stage * D::kStage;
    if (d < Cfg::A_DMA) {
      dma16_scalar_base(baseA + (size_t)s * kBlockBytes + d * Cfg::kWaves * 1024, lane * 16, dst + d * Cfg::kWaves * 1024);
    } else if (d < Cfg::A_DMA + D::X_DMA) {
      const int j = d - Cfg::A_DMA;
      const uint16_t* src = srcX[j] + (size_t)s * BK;
      // a piece beyond the end of the row (the padding of K; K is a multiple of 16) is filled with mask bytes: finite
      // numbers, and its weights are masked to zero
      if (s >= whole_slabs && s * BK + piece >= a.K) src = reinterpret_cast<const uint16_t*>(a.mask);
      dma16(src, lds0 + D::kRowsAt + stage * D::kRows + j * Cfg::kWaves * 1024);
    } else {
      const int j = d - Cfg::A_DMA - D::X_DMA;
      const int8_t* src = baseB + (size_t)s * kBlockBytes + j * Cfg::kWaves * 1024;
      const uint32_t to = dst + D::kCodes + j * Cfg::kWaves * 1024;
      if constexpr (kOnce) dma16_once(src + lane * 16, to);
      else dma16_scalar_base(src, lane * 16, to);
    }
  };
  auto fill_masks = [&](int s0) {
    const int words = min(D::kMaskSlabs, end - s0) * (BK / 4);
    for (int t = threadIdx.x; t < words; t += Cfg::kThreads)
      reinterpret_cast<uint32_t*>(s_mask)[t] = reinterpret_cast<const uint32_t*>(a.mask + (size_t)s0 * BK)[t] * 0xffu;   // bytes of 0 or 1
  };

  struct Frags {
    v4i x[TI], w[TJ];        // codes of both sides, one k-step
    v4u xf[2][TI], mk;       // rows of X, the two halves of the k-step; 0xff per critical column
  };
  const int a_off = (p.wm * Cfg::WM / 32) * 2048 + lane * 16;
  const int b_off = D::kCodes + (p.wn * Cfg::WN / 32) * 2048 + lane * 16;
  int x_off[TI];
#pragma unroll
  for (int i = 0; i < TI; ++i) x_off[i] = D::kRowsAt + (p.wm * Cfg::WM + i * 32 + p.lr) * (BK * 2);
  // read n (0 .. kReads - 1) of the fragments of k-step ks of slab s, in the order in which they are needed
  constexpr int kReads = TI + TJ + 1 + 2 * TI, kInt = TI * TJ, kAll = 3 * kInt;
  auto read_frag = [&](int s, int stage, int ks, Frags& f, int n) __attribute__((always_inline)) {
    const int8_t* base = smem + stage * D::kStage;
    if (n == 2) {
      f.mk = *reinterpret_cast<const v4u*>(s_mask + ((s - first) % D::kMaskSlabs) * BK + (2 * ks + p.lg) * 16);
    } else if (n < TI + TJ + 1) {
      const int e = n > 2;
      if (n == 0 || n == 3)
        f.x[e] = *reinterpret_cast<const v4i*>(base + a_off + e * 2048 + ks * 1024);
      else
        f.w[e] = *reinterpret_cast<const v4i*>(base + b_off + e * 2048 + ks * 1024);
    } else {
      const int t = (n - TI - TJ - 1) / TI, i = (n - TI - TJ - 1) % TI;
      const int q = 4 * ks + 2 * p.lg + t;                             // columns 8 q .. 8 q + 8 of the slab
      f.xf[t][i] = *reinterpret_cast<const v4u*>(smem + stage * D::kRows + x_off[i] + ((q ^ (p.lr >> 1 & 7)) * 16));
    }
  };
  static_assert(TI == 2 && (TJ == 2 || TJ == 1), "the orders of reads, conversions and MFMAs are written for 2 x 2 and 2 x 1 tiles");

  // ... those between MFMA n and the next: one, or two where there are more reads than MFMAs
  auto reads = [&](int n, int s, int stage, int ks, Frags& f) __attribute__((always_inline)) {
    constexpr int kTwice = kReads > kAll ? kReads - kAll : 0;
#pragma unroll
    for (int q = n + (n < kTwice ? n : kTwice); q < n + 1 + (n + 1 < kTwice ? n + 1 : kTwice); ++q)
      if (q < kReads) read_frag(s, stage, ks, f, q);
  };

  v16i acc[TI][TJ];
  v16f accf[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0, accf[i][j][e] = 0.0f;

  Frags f[2];
  // In iteration s slab s + 2 is requested into the buffer of slab s - 1, which every wave finished reading before the
  // barrier of iteration s - 1; past the end the last slab is asked for again, so that the count in flight is fixed.
  // One k-step: 12 (or 6) MFMAs, and between any two of them one fragment read of the next k-step (or two), the conversion of four
  // weight codes (ahead of their MFMA by as many as there are tiles) and at times a request, fenced so that they stay there: a
  // wave issues in order, and a burst of reads that finds the LDS queue full holds up the MFMAs behind it (with the
  // reads in one go a slab took 1.05 us).
  auto multiply = [&](const Frags& g, auto&& between) __attribute__((always_inline)) {
    v2u wh[2 * TJ][2];
#pragma unroll
    for (int n = 0; n < kAll; ++n) {
      if (n < kInt) {
        const int i = n & 1, j = n >> 1;
        acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(g.x[i], g.w[j], acc[i][j], 0, 0, 0);
      } else {
        const int c = (n - kInt) >> 1, t = c / TJ, j = c % TJ, i = n & 1;
        const v4u h = v4u{wh[c][0][0], wh[c][0][1], wh[c][1][0], wh[c][1][1]};
        accf[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(v8h, g.xf[t][i]), __builtin_bit_cast(v8h, h), accf[i][j], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      between(n);
      if (n < 4 * TJ) {
        const int c = n >> 1, t = c / TJ, j = c % TJ, d = n & 1;
        wh[c][d] = codes_to_half4(((uint32_t)g.w[j][2 * t + d] & g.mk[2 * t + d]) ^ 0x80808080u);   // other columns: zero
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // (a second tile of this workgroup, or requests of another kind of tile: LDS is free only then)
  if (!early) asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" : : : "memory");
  // the codes of two slabs, as far as they are not on their way, then the rows: slab `first` is there but for the newest X_DMA
  const int on_their_way = early ? early_slabs(end - first) : 0;
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (q >= on_their_way) {
#pragma unroll
      for (int d = 0; d < D::kPerSlab; ++d)
        if (d < Cfg::A_DMA || d >= Cfg::A_DMA + D::X_DMA) request(min(first + q, last), q, d);
    }
#pragma unroll
  for (int q = 0; q < 2; ++q)
#pragma unroll
    for (int d = Cfg::A_DMA; d < Cfg::A_DMA + D::X_DMA; ++d) request(min(first + q, last), q, d);
  fill_masks(first);
  wait_slab_and_sync<D::X_DMA>();
#pragma unroll
  for (int n = 0; n < kReads; ++n) read_frag(first, 0, 0, f[0], n);
  int stage = 0, s = first;
  for (int s0 = first + D::kMaskSlabs;; s0 += D::kMaskSlabs) {
    for (; s < min(s0, end); ++s) {
      const int stage1 = stage == 2 ? 0 : stage + 1, stage2 = stage1 == 2 ? 0 : stage1 + 1;
      multiply(f[0], [&](int n) __attribute__((always_inline)) {
        reads(n, s, stage, 1, f[1]);
        // the requests of slab s + 2
        const int d = n * D::kPerSlab / kAll;
        if (d < D::kPerSlab && (d * kAll + D::kPerSlab - 1) / D::kPerSlab == n) request(min(s + 2, last), stage2, d);
      });
      multiply(f[1], [&](int n) __attribute__((always_inline)) {
        // slab s + 1 has landed for every wave
        if (n == 0) wait_slab_and_sync<D::kPerSlab>();
        reads(n, min(s + 1, last), stage1, 0, f[0]);
      });
      stage = stage1;
    }
    if (s0 >= end) break;
    // (a loop of its own: with the loads of the masks inside it the compiler waited for every request in flight at the
    // end of each slab)
    __syncthreads();                                                   // every wave has read the masks so far
    fill_masks(s0);
    __syncthreads();
    read_frag(s0, stage, 0, f[0], 2);
  }
  asm volatile("s_waitcnt vmcnt(0)" : : : "memory");                   // the requests repeated past the end

  float cs[TJ], bn[TJ];
  ColumnTerms<Cfg>(a, p).use(cs, bn);
  if (a.tap_acc) {
    if (a.splits > 1)
      tap_accumulators<Cfg, true>(a, p, acc);
    else
      tap_accumulators<Cfg, false>(a, p, acc);
  }
  float step[TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j) step[j] = a.c[min(p.nw + j * 32 + p.lr, a.N - 1)] / 127.0f;
#pragma unroll
  for (int i = 0; i < TI; ++i) {
    float rm[16];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const v4f v = *reinterpret_cast<const v4f*>(a.r + p.mw + i * 32 + 8 * q + 4 * p.lg);
      rm[4 * q] = v[0], rm[4 * q + 1] = v[1], rm[4 * q + 2] = v[2], rm[4 * q + 3] = v[3];
    }
#pragma unroll
    for (int j = 0; j < TJ; ++j) {
      v16f y;
#pragma unroll
      for (int e = 0; e < 16; ++e) y[e] = (float)acc[i][j][e] * (rm[e] * cs[j]) + accf[i][j][e] * step[j];
      acc[i][j] = __builtin_bit_cast(v16i, y);
    }
  }
  // an adapter's low-rank operands: at most two slabs, straight from where they were prepared
  for (int fs = a.crit_slabs; fs < (split == a.splits - 1 ? a.f_slabs : 0); ++fs) {
    const int8_t* xs = reinterpret_cast<const int8_t*>(a.Xo) + ((size_t)(p.mw >> 8) * a.f_slabs + fs) * kBlockBytes + (p.mw & 255) * BK + lane * 16;
    const int8_t* ws = reinterpret_cast<const int8_t*>(a.Wo) + ((size_t)(p.nw >> 8) * a.f_slabs + fs) * kBlockBytes + (p.nw & 255) * BK + lane * 16;
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      v8h xa[TI], wb[TJ];
#pragma unroll
      for (int i = 0; i < TI; ++i) xa[i] = *reinterpret_cast<const v8h*>(xs + i * 2048 + ks * 1024);
#pragma unroll
      for (int j = 0; j < TJ; ++j) wb[j] = *reinterpret_cast<const v8h*>(ws + j * 2048 + ks * 1024);
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
          acc[i][j] = __builtin_bit_cast(v16i, __builtin_amdgcn_mfma_f32_32x32x16_f16(xa[i], wb[j], __builtin_bit_cast(v16f, acc[i][j]), 0, 0, 0));
    }
  }
  if (a.splits > 1)
    store_partial<Cfg>(a, p, acc, split);
  else if (a.codes || a.residual || a.gelu)
    store_tile_coded<Cfg, false>(a, p, acc, bn, smem, wave);
  else
    store_tile<Cfg, false>(a, p, acc, bn, smem, wave);
}

// ... over the 128-row pieces of the kernel's BM x BN tile.  The walk is part of the kernel's body, and reads the kernel's
// arguments through an address that the compiler cannot see through, where they are needed: what it computes from them is then
// not shared with the other way through the kernel, whose registers it would take.  (As a function of its own it saved and restored 120
// registers a lane through scratch, 24 to 63 MB of writes a launch.)  The address of the LDS buffers is handed on as a number: named,
// it would be read from memory again for every use.  Where the tile is walked in pieces, on the 256 x 256 tiles and configuration 2, the
// kernel still keeps 20 to 44 bytes a lane in scratch: the loops over pieces around the walk, its epilogue and, on 256 x 256 tiles, the
// gathering of columns beyond the slabs use them; the loops over slabs have no access to scratch.
template <class Cfg, bool kOnce>
__device__ __forceinline__ void gemm_tile_dense(const GemmArgs& a, int8_t* smem) {
  constexpr int kBN = Cfg::BN;
  constexpr bool kSameTile = std::is_same_v<Cfg, typename DenseCfg<kBN>::Tile>;
  int tm, tn, split;
  if (!tile_of_block(a, blockIdx.x, tm, tn, split)) return;
  if constexpr (kSameTile) {
    dense_tile<kBN, kOnce>(a, tm * Cfg::BM, tn * Cfg::BN, split, smem, true);
  } else {
    for (int n0 = tn * Cfg::BN; n0 < min((tn + 1) * Cfg::BN, a.N); n0 += kBN)
      for (int m0 = tm * Cfg::BM; m0 < min((tm + 1) * Cfg::BM, a.M); m0 += 128) dense_tile<kBN, kOnce>(a, m0, n0, split, smem, false);
  }
}

template <class Cfg>
using DenseOf = DenseCfg<Cfg::BN>;
// LDS of a launch: also the walk's (registers already keep a second workgroup off the compute unit)
template <class Cfg>
constexpr int kMostLds = Cfg::LDS_BYTES > DenseOf<Cfg>::LDS_BYTES ? Cfg::LDS_BYTES : DenseOf<Cfg>::LDS_BYTES;

// kOnce: the weights requested as bytes that nothing else reads (weights_read_once)
template <class Cfg, bool kTap, bool kFull, bool kCoded, bool kSplit, bool kOnce>
__global__ __launch_bounds__(Cfg::kThreads, Cfg::kWavesPerSimd) void k_gemm_mixed(const GemmArgs a) {
  extern __shared__ __attribute__((aligned(1024))) int8_t smem[];
  using constant_bytes = const __attribute__((address_space(4))) char*;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  int tm, tn, split;
  if (!tile_of_block(a, blockIdx.x, tm, tn, split)) return;           // (workgroup 0 always has a tile)
  const WavePos<Cfg> p(tm * Cfg::BM, tn * Cfg::BN, wave, threadIdx.x & (kWave - 1));
  const int first = kSplit ? split * a.slabs_per_split : 0;
  const int n_slabs = kSplit ? min(a.slabs_per_split, a.Kpad / BK - first) : a.Kpad / BK;
  const CodeRequests<Cfg, kOnce> codes_of(a, p, wave, first, (uint32_t)(uintptr_t)smem);
  // The first slabs, which both ways begin with, ahead of the count of critical columns and of the columns' scales: one after
  // the other, each a memory latency, they held the first product back: 2.4 us from a workgroup's start to it, 1.9 now (ViT-L
  // block of 1576 rows 111.9 -> 109.4 us, 7B-shaped layer of 256 heavy-tailed rows 242 -> 237).
#pragma unroll
  for (int q = 0; q < 2; ++q)
    if (q < early_slabs(n_slabs)) {
#pragma unroll
      for (int d = 0; d < Cfg::DMA_PER_SLAB; ++d) codes_of.issue(q, q, d);
    }
  // (through the scalar cache, so that the wait for it is not one for the requests; an address that the compiler cannot see
  // through keeps the load behind them)
  uint64_t count_at = reinterpret_cast<uint64_t>(a.n_out);
  asm volatile("" : "+s"(count_at));
  const int n_out = *(const __attribute__((address_space(4))) int*)(constant_bytes)count_at;
  reset_column_flags(a.flag_reset, a.Kpad);
  if (dense_critical_path(n_out, a.crit_slabs, a.dense_from, a.W_master != nullptr)) {
    uint64_t address = (uint64_t)(const char*)__builtin_amdgcn_kernarg_segment_ptr();   // `a` is the first argument
    uint32_t lds = (uint32_t)(uintptr_t)smem;
    asm volatile("" : "+s"(address), "+s"(lds));
    gemm_tile_dense<Cfg, kOnce>(*(const GemmArgs*)(constant_bytes)address, (int8_t*)(__attribute__((address_space(3))) int8_t*)lds);
    return;
  }
  gemm_tile<Cfg, kTap, kFull, kCoded, kSplit, kOnce>(a, p, wave, split, n_slabs, n_out, codes_of);
}

// ------------------------------------------------------------------------------------------------
// The kernels need more LDS than a kernel gets by default; the attribute is set once per instantiation and device,
// by prepare_gemm_kernels() (called when a workspace is set up) or else by the first launch.
template <class Cfg, bool kTap, bool kFull, bool kCoded, bool kSplit = false, bool kOnce = false>
static hipError_t ensure_lds_attribute() {
  // per device: the attribute belongs to the device's code object.  Two threads may both find it unset and set
  // it twice, which is harmless.
  static std::atomic<bool> attr_set[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
  if (attr_set[dev]) return hipSuccess;
  const void* fn = reinterpret_cast<const void*>(&k_gemm_mixed<Cfg, kTap, kFull, kCoded, kSplit, kOnce>);
  const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, kMostLds<Cfg>);
  if (e == hipSuccess) attr_set[dev] = true;
  return e;
}

template <class Cfg, bool kTap, bool kFull, bool kCoded, bool kSplit = false, bool kOnce = false>
static hipError_t launch_one(const GemmArgs& a, hipStream_t stream) {
  if (hipError_t e = ensure_lds_attribute<Cfg, kTap, kFull, kCoded, kSplit, kOnce>(); e != hipSuccess) return e;
  const int grid = ceil_div(a.tiles_m * a.tiles_n * a.splits, 8) * 8;
  hipLaunchKernelGGL((k_gemm_mixed<Cfg, kTap, kFull, kCoded, kSplit, kOnce>), dim3(grid), dim3(Cfg::kThreads), kMostLds<Cfg>, stream, a);
  return hipGetLastError();
}

// K in ranges
template <class Cfg>
static hipError_t launch_split(GemmArgs a, bool once, hipStream_t stream) {
  a.tiles_m = ceil_div(a.M, Cfg::BM);
  a.tiles_n = ceil_div(a.N, Cfg::BN);
  return a.tap_acc ? launch_one<Cfg, true, false, false, true>(a, stream)
         : once    ? launch_one<Cfg, false, false, false, true, true>(a, stream)
                   : launch_one<Cfg, false, false, false, true>(a, stream);
}
template <class Cfg>
static hipError_t prepare_split() {
  hipError_t e = ensure_lds_attribute<Cfg, true, false, false, true>();
  if (e == hipSuccess) e = ensure_lds_attribute<Cfg, false, false, false, true>();
  if (e == hipSuccess) e = ensure_lds_attribute<Cfg, false, false, false, true, true>();
  return e;
}

template <class Cfg, bool kOnce>
static hipError_t launch_output(const GemmArgs& a, bool full, hipStream_t stream) {
  if (a.codes || a.residual || a.gelu)
    return full ? launch_one<Cfg, false, true, true, false, kOnce>(a, stream) : launch_one<Cfg, false, false, true, false, kOnce>(a, stream);
  return full ? launch_one<Cfg, false, true, false, false, kOnce>(a, stream) : launch_one<Cfg, false, false, false, false, kOnce>(a, stream);
}
template <class Cfg>
constexpr bool kHasOnce = std::is_same_v<Cfg, Cfg0> || std::is_same_v<Cfg, Cfg5>;
template <class Cfg>
static hipError_t launch_cfg(GemmArgs a, hipStream_t stream, bool once = false) {
  a.tiles_m = ceil_div(a.M, Cfg::BM);
  a.tiles_n = ceil_div(a.N, Cfg::BN);
  a.splits = 1;
  a.slabs_per_split = a.Kpad / BK;
  const bool full = (a.M % Cfg::BM == 0) && (a.N % Cfg::BN == 0), coded = a.codes || a.residual || a.gelu;
  if (a.codes && Cfg::BN % (1 << a.code_log_block) != 0) return hipErrorInvalidValue;   // a block would leave the tile
  if (a.tap_acc) return coded ? launch_one<Cfg, true, false, true>(a, stream) : launch_one<Cfg, true, false, false>(a, stream);
  if constexpr (kHasOnce<Cfg>)
    if (once) return launch_output<Cfg, true>(a, full, stream);
  return launch_output<Cfg, false>(a, full, stream);
}

// every instantiation launch_cfg can reach
template <class Cfg, bool kOnce>
static hipError_t prepare_output() {
  hipError_t e = ensure_lds_attribute<Cfg, false, true, false, false, kOnce>();
  if (e == hipSuccess) e = ensure_lds_attribute<Cfg, false, false, false, false, kOnce>();
  if (e == hipSuccess) e = ensure_lds_attribute<Cfg, false, true, true, false, kOnce>();
  if (e == hipSuccess) e = ensure_lds_attribute<Cfg, false, false, true, false, kOnce>();
  return e;
}
template <class Cfg>
static hipError_t prepare_cfg() {
  hipError_t e = ensure_lds_attribute<Cfg, true, false, false>();
  if (e == hipSuccess) e = ensure_lds_attribute<Cfg, true, false, true>();
  if (e == hipSuccess) e = prepare_output<Cfg, false>();
  if constexpr (kHasOnce<Cfg>)
    if (e == hipSuccess) e = prepare_output<Cfg, true>();
  return e;
}
hipError_t prepare_gemm_kernels() {
  hipError_t e = prepare_cfg<Cfg0>();
  if (e == hipSuccess) e = prepare_cfg<Cfg1>();
  if (e == hipSuccess) e = prepare_cfg<Cfg2>();
  if (e == hipSuccess) e = prepare_cfg<Cfg3>();
  if (e == hipSuccess) e = prepare_cfg<Cfg4>();
  if (e == hipSuccess) e = prepare_cfg<Cfg5>();
  if (e == hipSuccess) e = prepare_split<Cfg0>();
  if (e == hipSuccess) e = prepare_split<Cfg5>();
  return e;
}

static hipError_t launch_variant(const GemmArgs& a, int variant, hipStream_t stream, bool once = false) {
  // coded output with blocks wider than the 128-column tiles
  if (a.codes && a.code_log_block > 7 && variant <= 1) variant = 5;
  switch (variant) {
    case 1: return launch_cfg<Cfg1>(a, stream);
    case 2: return launch_cfg<Cfg2>(a, stream);
    case 3: return launch_cfg<Cfg3>(a, stream);
    case 4: return launch_cfg<Cfg4>(a, stream);
    case 5: return launch_cfg<Cfg5>(a, stream, once);
    default: return launch_cfg<Cfg0>(a, stream, once);
  }
}

// the same problem restricted to output columns [n0, n0 + n): n0 a multiple of 256
static GemmArgs column_range(const GemmArgs& a, int n0, int n) {
  GemmArgs b = a;
  const size_t panels = (size_t)n0 / kPanelRows;
  b.Wt = a.Wt + panels * (size_t)(a.Kpad / BK) * kBlockBytes;
  b.Wo = a.Wo + panels * a.f_slabs * (kBlockBytes / 2);            // uint16_t elements
  b.Wg = a.Wg ? a.Wg + panels * a.g_slabs * (kBlockBytes / 2) : nullptr;
  b.c = a.c + n0;
  b.bias = a.bias ? a.bias + n0 : nullptr;
  b.Y = a.Y ? a.Y + n0 : nullptr;
  b.residual = a.residual ? a.residual + n0 : nullptr;
  b.codes = a.codes ? a.codes + n0 : nullptr;
  b.code_absmax = a.codes ? a.code_absmax + (n0 >> a.code_log_block) : nullptr;   // n0 is a multiple of 256
  b.tap_acc = a.tap_acc ? a.tap_acc + n0 : nullptr;
  b.W_master = a.W_master ? a.W_master + n0 : nullptr;
  b.N = n;
  return b;
}

// 128 x 128 tiles (of `splits` ranges of K) that fit in one round.  Ranges go on such tiles wherever they do, else on 128 x 256:
// at the same count of ranges the small tiles measured faster in 2309 of 2321 pairs.
bool one_round_of_small_tiles(int M, int N, int splits) { return (long)ceil_div(M, 128) * ceil_div(N, 128) * splits <= device_cu_count(); }
int plan_gemm_splits(int M, int K, int N) {
  const int n_slabs = packed_k(K) / BK, cus = device_cu_count();
  const long tiles = (long)ceil_div(M, Cfg5::BM) * ceil_div(N, Cfg5::BN);
  if (M <= 128 || 2 * tiles > cus) return 1;
  // The cost of s ranges: the slabs of a workgroup, the launch that adds the ranges up, and the sums.  The constants are
  // fitted to the choice and not to the time: 950 calls (129 to 2600 rows, K 512 to 16384, N 256 to 8192), each without a split and
  // with up to 24 ranges of either tile, weights from memory and still in the last-level cache, where a split gains less, few critical
  // columns and heavy-tailed rows, where it gains more (the walk with both products takes twice as long per slab); the host cannot
  // tell these apart.  Over these calls the count taken is 1.3 % slower than the best one with few critical columns and weights from
  // memory, 2.4 % with cached ones, 4.1 and 3.2 % with heavy-tailed rows; at worst 45 %, where K of 600 to 1500 is not split.  Us, few
  // and heavy-tailed, weights from memory, without a split / as taken / other ranges: 333 x 4096 x 4096 31.1 and 51.8 / 27.6 and 39.7
  // (2) / 29.8 and 40.0 (4 of 128 x 256 tiles); 256 x 4096 x 4096 30.6 and 49.9 / 25.6 and 32.5 (3) / 27.5 and 32.3 (4); 247 x 2400 x
  // 880 22.3 and 34.3 / 17.7 and 21.1 (5) / 20.1 and 24.8 (6 of 128 x 256); 175 x 3296 x 1352 25.8 and 40.7 / 19.3 and 22.8 (6) / 23.7
  // and 26.7 (12 of 128 x 256); 175 x 3440 x 5648 27.7 and 44.0 / 25.7 and 34.0 (2) / 27.0 and 34.7 (4 of 128 x 256); 256 x 11008 x 4096
  // 61.3 and 112.8 / 38.2 and 56.0 (4) / 43.0 and 56.7 (8 of 128 x 256); 333 x 11008 x 4096 61.5 and 138.8 / 43.2 and 97.2 (5 of 128 x
  // 256) / 45.2 and 102.7 (2).  No split taken: 400 x 2048 x 2048 20.7 and 30.8, with two ranges 21.6 and 27.4.
  // (The term of the sums is the same for both tiles, so that the count falls as M grows within a row of tiles:
  // linear_workspace_bytes relies on it.)
  int best = 1;
  double least = (one_round_of_small_tiles(M, N) ? 0.2551 : 0.1277) * n_slabs;
  for (int s = 2; s * tiles <= cus && n_slabs / s >= 4; ++s) {
    const int slabs = ceil_div(n_slabs, s);
    const double cost = (one_round_of_small_tiles(M, N, s) ? 4.44 + 0.2185 * slabs : 3.972 + 0.281 * slabs) + 1.4555e-6 * s * M * N;
    if (cost < least) best = s, least = cost;
  }
  return ceil_div(n_slabs, ceil_div(n_slabs, best));
}

// Where the line between slabs and dense_tile lies.  The walk with both products costs the same whatever their number: more than
// the walk over the codes by an amount that grows with the slabs of a range, on 128 x 256 tiles and taller ones also with the rounds of
// tiles, and where the ranges leave fp32 sums, with those.  The slabs cost their preparation, whose first microseconds are the
// offset, and per column a place in the ring, so that beyond two thirds of a range's columns (`most`) the walk is never the dearer
// one; a column beyond the slabs is gathered tile by tile.  The constants are fitted to the choice: 1201 calls (129 to 4096 rows,
// K 288 to 16384 and 32768, N 256 to 22016; split, and without the split that a small workspace has no room for; weights from memory and, a
// fifth of them, still in the last-level cache), each measured both ways with 3 to 97 % of the columns critical.  With weights from memory
// the way taken is 0.4 % slower than the better one on average (the line fitted to the kernels before these 3.0 %, for split calls
// 5.6), more than 10 % in one of ninety, at worst 33 % where it is the slabs (163 x 15040 x 20848 at 17 %) and 21 % where it is the
// walk (2059 x 4816 x 1744 at 28 %).  Whole calls, us, walk / slabs: 256 x 4096 x 4096 33.0 / 38.0 at 7.5 %, not split 48.7 / 46.5 at 10 %,
// 48.9 / 52.2 at 13 %; 256 x 11008 x 4096 48.8 / 59.6 at 5 %; 333 x 4096 x 22016 135 / 117 at 22 %, 136 / 154 at 36 %; 2048 x 4096 x
// 12288 293 / 263 at 46 %, 298 / 350 at 60 %; 2048 x 1024 x 4096 66 / 64 at 60 %, 66 / 74 at 80 %; 4096 x 8192 x 10240 855 / 563 at
// 28 %, 866 / 924 at 36 %.
CriticalPlan plan_critical_columns(int M, int n_slabs, int N, bool further_slabs, int splits) {
  CriticalPlan p = {0, 0};
  const size_t Npad = packed_n(N);
  if (further_slabs) {
    size_t cols = (size_t)n_slabs * 32;                              // half of the columns at most
    if (cols > (size_t)kGatherMax) cols = kGatherMax;
    const size_t fit = kGatherWeightBytesMax / (Npad * 2);
    if (cols > fit) cols = fit;
    p.g_slabs = (int)(cols / kOutlierSlab);
  }
  const int in_slabs = kOutlierSlab * (kCriticalSlabs + p.g_slabs);
  const double rounds = (double)ceil_div(M, 128) * ((double)Npad / 256) / device_cu_count();   // of 128 x 256 tiles
  const int slabs = ceil_div(n_slabs, splits);
  const double per_slab = one_round_of_small_tiles(M, N, splits) ? 9.6 : 13.0 + 6.7 * rounds, most = slabs * BK * (0.64 + 0.09 * rounds);
  double from = 0.475 * M + per_slab * slabs - 360.0;
  if (splits > 1) from += 27e-6 * splits * M * (double)Npad;
  if (from > most) from = most;
  if (from > in_slabs) from = in_slabs + (from - in_slabs) * (0.144 + 0.072 * rounds) / (rounds > 1 ? rounds : 1);
  p.dense_from = from < 1e9 ? (int)from : 1000000000;
  return p;
}

// Weights requested as bytes that nothing else reads leave the last-level cache (256 MB) to the rest of a layer: for up to
// four rows of tiles, and for matrices so large that the model they belong to does not stay in that cache.  Us per
// layer of four linears (weights from memory but for hidden size 1536 and less), few critical columns, with plain / such
// requests: hidden size 3072, 256 rows 152 / 140; 4096, 129 rows 168 / 156; 5120, 333 rows 234 / 234.  For every matrix from
// 9 MB on: hidden size 1536 87 / 91 us at 333 rows, 2048 93 / 101 at 129 rows (from 22 MB on 92), and a call of 512 x 4096 ->
// 4096 whose weights are in the cache 33 / 41.  More rows: 768 x 4096 -> 22016 106 / 110, 1024 x 28672 -> 8192 244 / 256.
// (A choice between the two inside the kernel cost the walk 2 %: two instantiations.)
bool weights_read_once(int M, int Kpad, int N) { return M > 128 && M <= 512 && (size_t)Kpad * N >= 20000000; }

hipError_t launch_gemm_mixed(GemmArgs a, int variant, hipStream_t stream) {
  if (variant >= 0 && variant <= 5) return launch_variant(a, variant, stream);
  const bool once = weights_read_once(a.M, a.Kpad, a.N);
  if (a.partial && a.splits > 1) {
    const int n_slabs = a.Kpad / BK;
    a.slabs_per_split = ceil_div(n_slabs, a.splits);
    if (ceil_div(n_slabs, a.slabs_per_split) != a.splits) return hipErrorInvalidValue;   // every range has a slab
    hipError_t e = hipSuccess;
    if (a.tap_acc) e = launch_fill_u32(reinterpret_cast<uint32_t*>(a.tap_acc), 0u, (size_t)a.M * a.tap_ld, stream);
    if (e == hipSuccess) e = one_round_of_small_tiles(a.M, a.N, a.splits) ? launch_split<Cfg0>(a, once, stream) : launch_split<Cfg5>(a, once, stream);
    if (e != hipSuccess) return e;
    const SplitSum sum = {a.partial, a.splits, a.M, a.N, a.bias, a.residual, a.ldr, a.gelu, a.Y, a.ldy,
                          a.codes, a.code_absmax, a.codes ? 1 << a.code_log_block : 0};
    return launch_add_splits(sum, stream);
  }
  // Automatic.  The 256 x 256 tile with the four-slab ring is the most efficient per CU, but it runs
  // in rounds of one tile per CU.  Whole rounds go to it; a remainder that would leave a good part of
  // the chip idle is launched separately with 128 x 256 tiles (same ring depth, twice as many
  // workgroups).  With weights coming cold from HBM (every layer has its own) the deep prefetch
  // matters more than the better balance of small tiles, so small tiles are for small problems only.
  const int tiles_m = ceil_div(a.M, 256), tiles_n = ceil_div(a.N, 256);
  const long tiles_256 = (long)tiles_m * tiles_n;
  const long tiles_128x256 = (long)ceil_div(a.M, 128) * tiles_n;
  const long cus = device_cu_count();
  if (a.M > 128 && tiles_256 >= cus) {
    const long rest = tiles_256 % cus;
    const int n_tiles_main = (int)((tiles_256 - rest) / tiles_m);      // whole columns of tiles in the whole rounds
    const int n_tiles_rest = tiles_n - n_tiles_main;
    if (rest > 0 && 2 * rest <= cus && n_tiles_main > 0 && n_tiles_rest > 0) {
      hipError_t e = launch_variant(column_range(a, 0, n_tiles_main * 256), 4, stream);
      if (e != hipSuccess) return e;
      return launch_variant(column_range(a, n_tiles_main * 256, a.N - n_tiles_main * 256), 5, stream);
    }
    return launch_variant(a, 4, stream);
  }
  // Less than one round of large tiles: 128 x 128 tiles where they fit one round, else 128 x 256 with eight waves and the
  // four-slab ring.  (Measured, the kernel alone, 128 x 128 / 128 x 256: 256 x 4096 x 12288 21.0 / 28.6 us, 1000 x 4096 x 4096
  // 24.0 / 30.1, 1024 x 1024 x 4096 12.6 / 14.0; whole calls, the former still with four waves, 300 x 4096 x 12288, where the small
  // tiles are a round and a bit, 52 / 39.)  Where the 128 x 256
  // tiles would need a second round and the 256 x 256 ones fit in one, the large tiles win: 4096 -> 12288 at 768 rows 61
  // against 71 us, 4096 -> 22016 at 512 rows 61 against 70.
  if (a.M > 128 && tiles_128x256 > cus) return launch_variant(a, 4, stream);
  if (a.M > 64 && !one_round_of_small_tiles(a.M, a.N)) return launch_variant(a, 5, stream, once);
  return launch_variant(a, 0, stream, once);
}

}  // namespace mmd8
