// bf16 MFMA GEMM tile for gfx950: D[256 x 256] (fp32) = A[256 x K] * B[256 x K]^T, both
// operands row-major with K contiguous.  One workgroup of 8 waves (2 x 4, two per SIMD) owns
// the tile; each wave accumulates a 128 x 64 sub-tile as 8 x 4 blocks of
// v_mfma_f32_16x16x32_bf16.  Two waves per SIMD let one wave's waits (barrier, LDS latency,
// epilogue arithmetic) hide behind the other's matrix instructions.
//
// Two things bound the loop, in about equal parts.  The power limit: k_fused_stats<false> at 151936 x 16384 x 1536 takes
// 5.92 ms on Gaussian operands at 1.97 GHz and 4.95 on zeros at 2.39, the matrix units busy in 62 % of the cycles both
// times, so the energy per flop of the matrix instruction counts; a stream of nothing but 16 x 16 x 32 reaches 2.11
// PFLOP/s on Gaussian data where 32 x 32 x 16 reaches 1.85 (both 2.4-2.5 on zeros), and 2.13 when consecutive
// instructions always share one operand (the column order alternates from row to row).  And the other 38 % of the
// cycles, part of which the clock would take back: the library's 81 % at K = 3584 come with 1.70 GHz.  The bare loop below:
// 1.45 PFLOP/s at 151936 x 16384 x 1536 and 1.44 at 152064 x 32768 x 3584, against 1.36 / 1.34 with 32 x 32 x 16.
//
// Two main loops share the accumulator layout:
//   gemm_tile_dma  operands go HBM -> LDS directly (buffer_load ... lds), two stages of
//                  256 x 64 slices, L2 warmed two slices ahead; needs K % 64 == 0 and
//                  16-byte aligned rows
//   gemm_tile      register-staged 256 x 64 slices with explicit predication; any K % 8 == 0
#pragma once
#include "aero_device.h"

namespace aero {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int kTile = 256;          // tile edge in both output dimensions
constexpr int kGemmNT = 512;        // threads per workgroup (8 waves)
constexpr int kMB = 8, kNB = 4;     // 16 x 16 blocks per wave: 128 rows x 64 columns
constexpr size_t kGemmStageBytes = 131072;  // two stages of (256 + 256) x 64 bf16
constexpr size_t kWarmSinkOff = kGemmStageBytes;   // past the stages
constexpr size_t kGemmLdsBytes = kWarmSinkOff + 2048;   // + a 256-byte sink per wave for the warm-up loads

// Position of an accumulator element inside the 256 x 256 tile.
//   block (mb, nb) of wave (wm in 0..1, wn in 0..3); register i of lane l:
//   row = wm*128 + mb*16 + 4*(l/16) + i,   col = wn*64 + nb*16 + l%16
// SWAP (a template argument of the loops): the operands of the matrix instruction are exchanged, and
//   row = wm*128 + mb*16 + l%16,           col = wn*64 + nb*16 + 4*(l/16) + i
// i.e. a lane holds four consecutive columns of one row instead of four rows of one column.
__device__ __forceinline__ int acc_row(int wm, int mb, int i, int lane) { return wm * 128 + mb * 16 + 4 * (lane >> 4) + i; }
__device__ __forceinline__ int acc_col(int wn, int nb, int lane) { return wn * 64 + nb * 16 + (lane & 15); }
__device__ __forceinline__ int acc_row_swapped(int wm, int mb, int lane) { return wm * 128 + mb * 16 + (lane & 15); }
__device__ __forceinline__ int acc_col_swapped(int wn, int nb, int lane) { return wn * 64 + nb * 16 + 4 * (lane >> 4); }

// Which part of the tile a wave owns.  Waves w and w + 4 run on the same SIMD; the two that share one are the halves
// of the dimension that may be ragged, so that skipping waves whose rows or columns are all padding halves the work
// of every SIMD: rows of A (wave_pos<false>) or columns of B, in steps of two blocks of 64 (wave_pos<true>).
// Whole calls at H = 1536, V = 151936: 600 tokens (a third tile with 88) 905 -> 873 us, 1100 and 16384 tokens even;
// 1400 tokens at H = 3584, V = 32000 826 -> 815; 300 tokens at H = 896, V = 8000 102.2 -> 103.7.
struct WavePos {
  int wm, wn;
  bool active;   // false: all of the wave's rows (columns) are padding, its accumulators stay zero
};
template <bool RAGGED_COLS> __device__ __forceinline__ WavePos wave_pos() {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  return RAGGED_COLS ? WavePos{wave & 1, wave >> 1, true} : WavePos{wave >> 2, wave & 3, true};
}

typedef f32x4_t Acc[kMB][kNB];

__device__ __forceinline__ void acc_zero(Acc& acc) {
#pragma unroll
  for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) acc[mb][nb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
}

// Workgroup id -> tile.  Consecutive hardware workgroup ids go to different XCDs (8 of them,
// each with its own L2), so ids are first regrouped per XCD; inside that order tiles walk
// bands of 8 tile-rows so that concurrently resident workgroups share operand slices in L2.
// xcd_regroup: position of hardware workgroup `pid` (of `nb`) in the per-XCD contiguous order.
__device__ __forceinline__ int xcd_regroup(int pid, int nb) {
  const int q = nb / 8, r = nb % 8, xcd = pid % 8;
  return xcd * q + min(xcd, r) + pid / 8;
}

// npid in [0, tiles_m * tiles_n) -> tile, bands of 8 tile-rows, row index fastest inside a band
__device__ __forceinline__ void tile_of_index(int npid, int tiles_m, int tiles_n, int& tm, int& tn) {
  constexpr int GM = 8;
  const int group_sz = GM * tiles_n;
  const int first_m = (npid / group_sz) * GM;
  const int gm = min(GM, tiles_m - first_m);
  const int within = npid % group_sz;
  tm = first_m + within % gm;
  tn = within / gm;
}

// The same regrouping in whole columns of a band: the n positions of a launch are cut into units
// of 8 consecutive positions (one column of 8 tile rows), every XCD gets a contiguous run of
// whole units (run lengths differ by at most one unit), so that the workgroups resident on an
// XCD always cover whole columns, whatever n is.  The launch grid is xcd_grid(n) >= n workgroups;
// the surplus ones get -1 and leave.
inline int xcd_grid(int n) { return 64 * (((n + 7) / 8 + 7) / 8); }
__device__ __forceinline__ int xcd_position(int pid, int n) {
  const int units = (n + 7) / 8, q = units / 8, r = units % 8;
  const int xcd = pid % 8, local = pid / 8;
  const int ul = local / 8;
  if (ul >= q + (xcd < r ? 1 : 0)) return -1;
  const int pos = (xcd * q + min(xcd, r) + ul) * 8 + local % 8;
  return pos < n ? pos : -1;
}

// tile0: position in the tile order of this launch's first tile, n: tiles of this launch (a
// kernel's tiles may be spread over several launches).  False: a surplus workgroup.
__device__ __forceinline__ bool tile_of_block(int tiles_m, int tiles_n, int tile0, int n, int& tm, int& tn) {
  const int pos = xcd_position(blockIdx.x, n);
  if (pos < 0) return false;
  tile_of_index(tile0 + pos, tiles_m, tiles_n, tm, tn);
  return true;
}

// Fragments of one 32-wide K step: lane l holds K 8 (l/16) .. + 7 of row l%16 of a 16-row block.
// A wave's 128 rows of A come in two halves of four blocks.
constexpr int kFragBlocks = 4;
typedef bf16x8_t Frags[kFragBlocks];

template <bool SWAP>
__device__ __forceinline__ void frags_mma(const Frags& a, const Frags& b, int half, Acc& acc) {
#pragma unroll
  for (int i = 0; i < kFragBlocks; ++i)
#pragma unroll
    for (int jj = 0; jj < kNB; ++jj) {
      const int j = (i & 1) ? kNB - 1 - jj : jj;   // neighbours in the sequence share an operand (see the top)
      f32x4_t& c = acc[half * kFragBlocks + i][j];
      c = SWAP ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], c, 0, 0, 0)
               : __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], c, 0, 0, 0);
    }
}

// ------------------------------------------------------------------------------------------
// Register-staged loop (fallback): 256 x 64 slices, double buffered, explicit predication.
// ------------------------------------------------------------------------------------------
constexpr int kBK = 64;
constexpr int kSliceElems = kTile * kBK;
static_assert(size_t(4) * kSliceElems * 2 <= kGemmStageBytes, "double buffer must fit the LDS budget");
constexpr int kVecPerThread = kTile * (kBK / 8) / kGemmNT;   // 4

__device__ __forceinline__ void slice_load(const uint16_t* __restrict__ base, int64_t ld, int row0,
                                           int rows_valid, int k0, int K, u32x4_t (&r)[kVecPerThread]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int v = 0; v < kVecPerThread; ++v) {
    const int idx = tid + v * kGemmNT;
    const int row = row0 + (idx >> 3), k = k0 + ((idx & 7) << 3);
    if (row < rows_valid && k < K)
      r[v] = *reinterpret_cast<const u32x4_t*>(base + int64_t(row) * ld + k);
    else
      r[v] = u32x4_t{0u, 0u, 0u, 0u};
  }
}

// Rows are 128 bytes; rows of equal parity share a 128-byte half of the 256-byte bank line, so
// the chunk index is swizzled with bits 1..3 of the row: 16 consecutive rows -> 16 distinct slots.
__device__ __forceinline__ int lds_off(int row, int chunk) {
  return row * kBK + ((chunk ^ ((row >> 1) & 7)) << 3);
}

__device__ __forceinline__ void slice_store(uint16_t* lds, const u32x4_t (&r)[kVecPerThread]) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int v = 0; v < kVecPerThread; ++v) {
    const int idx = tid + v * kGemmNT;
    *reinterpret_cast<u32x4_t*>(lds + lds_off(idx >> 3, idx & 7)) = r[v];
  }
}

// Fragments of K step ks (0, 1) of a 64-wide slice held in LDS: four 16-row blocks from row0 on.
__device__ __forceinline__ void frags_load(Frags& f, const uint16_t* lds, int row0, int ks, int lane) {
#pragma unroll
  for (int i = 0; i < kFragBlocks; ++i)
    f[i] = *reinterpret_cast<const bf16x8_t*>(lds + lds_off(row0 + i * 16 + (lane & 15), ks * 4 + (lane >> 4)));
}

template <bool SWAP>
__device__ __forceinline__ void slice_mma(const uint16_t* As, const uint16_t* Bs, int wm, int wn, int lane, Acc& acc) {
#pragma unroll
  for (int ks = 0; ks < kBK / 32; ++ks) {
    Frags a, b;
    frags_load(b, Bs, wn * 64, ks, lane);
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      frags_load(a, As, wm * 128 + half * 64, ks, lane);
      frags_mma<SWAP>(a, b, half, acc);
    }
  }
}

// Full K loop for one tile.  A rows [m0, m0+256) clipped to M, B rows [n0, n0+256) clipped to
// N, columns [0, K).  smem: kGemmLdsBytes.  Ends with a barrier: smem is free afterwards.
template <bool SWAP>
__device__ __forceinline__ void gemm_tile(const uint16_t* __restrict__ A, int64_t lda, int M,
                                          const uint16_t* __restrict__ B, int64_t ldb, int N, int K,
                                          int m0, int n0, const WavePos& pos, uint16_t* smem, Acc& acc) {
  const int lane = threadIdx.x & 63;
  const int wm = pos.wm, wn = pos.wn;
  acc_zero(acc);
  const int nk = (K + kBK - 1) / kBK;
  if (nk == 0) return;
  uint16_t* As[2] = {smem, smem + 2 * kSliceElems};
  uint16_t* Bs[2] = {smem + kSliceElems, smem + 3 * kSliceElems};
  u32x4_t ra[kVecPerThread], rb[kVecPerThread];
  slice_load(A, lda, m0, M, 0, K, ra);
  slice_load(B, ldb, n0, N, 0, K, rb);
  slice_store(As[0], ra);
  slice_store(Bs[0], rb);
  __syncthreads();
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    const bool more = kt + 1 < nk;
    if (more) {
      slice_load(A, lda, m0, M, (kt + 1) * kBK, K, ra);
      slice_load(B, ldb, n0, N, (kt + 1) * kBK, K, rb);
    }
    slice_mma<SWAP>(As[cur], Bs[cur], wm, wn, lane, acc);
    if (more) {
      slice_store(As[cur ^ 1], ra);
      slice_store(Bs[cur ^ 1], rb);
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------------------------------
// Direct-to-LDS loop.  buffer_load ... lds moves 16 bytes per lane from HBM/L2 straight into
// LDS (lane l of a wave lands at LDS base + 16 l): no staging registers, no LDS stores, and the
// buffer descriptor's bounds check turns rows past the operand's end into zeros.  Slices are
// 256 x 64: every row contributes one full 128-byte line per slice (32-wide slices fetch half
// lines and lose a tenth of the throughput), two stages of 64 KB.
//
// Completion of these loads is tracked by hand: vmcnt(0) at the top of an iteration means this
// wave's part of the slice has landed, the barrier then makes every wave's part visible and
// also guarantees that the other stage is no longer being read.  The compiler does not model
// these dependencies, hence the explicit waits and compiler fences.
// ------------------------------------------------------------------------------------------
constexpr int kDK = kBK;                         // K slice of the fast loop
constexpr int kDStageElems = 2 * kTile * kDK;    // A then B
static_assert(size_t(2) * kDStageElems * 2 <= kGemmStageBytes, "two stages must fit the LDS budget");

// An operand of the fast loop: rows of 64-wide K slices.  Element (row, k) lives at
//   base + (k / 64) * kstep + row * ld + k % 64
//   row-major [rows, K]:            ld = row pitch, kstep = 64
//   K-slab layout [K/64][rows][64]: ld = 64,        kstep = rows * 64  (a 256-row slice is one
//                                   contiguous 32 KB block: the layout of the library's own
//                                   intermediate operands)
// bytes bounds the buffer: loads past it return zeros.
struct DmaOperand {
  const uint16_t* base;
  int64_t ld, kstep, bytes;
};
__device__ __forceinline__ DmaOperand operand_row_major(const uint16_t* base, int64_t ld, int rows_valid, int K) {
  return DmaOperand{base, ld, kDK, rows_valid > 0 ? ((int64_t(rows_valid) - 1) * ld + K) * 2 : 0};
}
__device__ __forceinline__ DmaOperand operand_slabs(const uint16_t* base, int64_t rows, int K) {
  return DmaOperand{base, kDK, rows * kDK, int64_t(K / kDK) * rows * kDK * 2};
}
// K-slabs in fragment order (AF): inside a slab every 16 rows are one 2 KB block, the two 32-wide K steps one after
// the other, each as the 16 x 16 x 32 instruction's lanes hold it: element (row, k) at
//   (row / 16) * 1024 + (k % 64 / 32) * 512 + (k % 32 / 8) * 128 + (row % 16) * 8 + k % 8
// A wave's accumulators can be stored in it straight from registers, 1 KB per instruction, and a fragment is 1 KB of
// LDS read lane by lane.
__device__ __forceinline__ int64_t frag_order_offset(int64_t rows, int64_t row, int64_t k) {
  return (k / 64) * rows * 64 + (row / 16) * 1024 + (k % 64 / 32) * 512 + (k % 32 / 8) * 128 + (row % 16) * 8 + k % 8;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_rsrc(const DmaOperand& o) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(o.base), 0, int(o.bytes), 0x00020000);
}

#define AERO_CFENCE() asm volatile("" ::: "memory")

// Per-lane byte offsets of the DMA loads of one operand.  Wave w fills rows [32 w, 32 w + 32)
// with 4 instructions of 8 rows; lane l covers row l/8 of those 8 and LDS slot l%8, and the
// chunk that belongs in that slot is slot ^ ((row >> 1) & 7) with row = 32 w + 8 j + l/8, i.e.
// (l % 8) ^ ((4 j + l / 16) & 7): one offset for even j, one for odd j.
struct DmaLane {
  uint32_t even, odd, row_step, k_step;
};
__device__ __forceinline__ DmaLane dma_lane(int row0, const DmaOperand& o, int wave, int lane) {
  const uint32_t row = uint32_t((int64_t(row0 + wave * 32 + (lane >> 3)) * o.ld) * 2);
  const uint32_t c0 = uint32_t((lane & 7) ^ ((lane >> 4) & 7)), c1 = uint32_t((lane & 7) ^ ((4 + (lane >> 4)) & 7));
  return DmaLane{row + c0 * 16, row + c1 * 16, uint32_t(8 * o.ld * 2), uint32_t(o.kstep * 2)};
}

// The same for an operand in fragment order: a wave's 32 rows are 4 KB in one piece.
__device__ __forceinline__ DmaLane dma_lane_af(int row0, const DmaOperand& o, int wave, int lane) {
  const uint32_t at = uint32_t((row0 + wave * 32) * kDK * 2 + lane * 16);
  return DmaLane{at, at, 1024u, uint32_t(o.kstep * 2)};
}

// The whole byte offset travels in the vector offset: the hardware bounds check covers the
// vector offset only, not the scalar one.
__device__ __forceinline__ void dma_issue(__amdgpu_buffer_rsrc_t ra, __amdgpu_buffer_rsrc_t rb, const DmaLane& la,
                                          const DmaLane& lb, int kt, uint16_t* stage, int wave) {
  uint16_t* a_dst = stage + wave * 32 * kDK;
  uint16_t* b_dst = stage + kTile * kDK + wave * 32 * kDK;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, a_dst + j * 8 * kDK, 16,
                                             ((j & 1) ? la.odd : la.even) + uint32_t(kt) * la.k_step + j * la.row_step, 0, 0, 0);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, b_dst + j * 8 * kDK, 16,
                                             ((j & 1) ? lb.odd : lb.even) + uint32_t(kt) * lb.k_step + j * lb.row_step, 0, 0, 0);
  }
}

// An operand stored the other way round (BT): a row-major matrix whose rows are the contraction index, [K][rows],
// e.g. the weight in dhidden = dz weight.  A slice is 64 rows of 256 columns (512 bytes, whole lines again); its LDS
// image keeps that orientation, [64][256], and fragments come out of it with the transposing LDS read
// (ds_read_b64_tr_b16): of every 16 lanes, lane j names four consecutive columns 4 (j % 4) .. of row j / 4, and
// receives column j of those four rows, so two reads make the eight K values of a fragment.  The 32-byte
// segments of a row are XORed with f(row) = row % 4 + 4 ((row / 8) % 2): the eight rows that 32 lanes touch at once
// fall on distinct banks.
__device__ __forceinline__ DmaLane dma_lane_bt(int col0, int64_t ld, int wave, int lane) {
  // wave w fills rows [8 w, 8 w + 8) with 4 instructions of 2 rows; lane l covers chunk l % 32 of row l / 32
  const uint32_t row = uint32_t(int64_t(wave * 8 + (lane >> 5)) * ld * 2 + int64_t(col0) * 2) + uint32_t(lane & 1) * 16;
  const uint32_t seg = (lane & 31) >> 1, f = uint32_t(lane >> 5) | uint32_t(wave & 1) << 2;
  return DmaLane{row + (seg ^ f) * 32, row + (seg ^ (f | 2)) * 32, uint32_t(4 * ld), uint32_t(kDK * ld * 2)};
}
__device__ __forceinline__ void frags_load_bt(Frags& f, const uint16_t* lds, int col0, int ks, int lane) {
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
  const int group = lane >> 4, j = lane & 15;
  const int swz = (j >> 2) | (group & 1) << 2;
  const uint16_t* base = lds + (ks * 32 + group * 8 + (j >> 2)) * kTile + (j & 3) * 4;
#pragma unroll
  for (int i = 0; i < kFragBlocks; ++i) {
    const uint16_t* at = base + ((col0 / 16 + i) ^ swz) * 16;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)at);
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)(at + 4 * kTile));
    const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    f[i] = __builtin_bit_cast(bf16x8_t, both);
  }
}

// WARM: L2 warm-up two slices ahead (see below); a few per cent on the contractions whose
// operands come from large read-only arrays, a loss on the split-K dhidden contraction.
// BT: operand B is [K][rows] (B.base, B.ld, B.bytes; B.kstep is not looked at).  AF: operand A is in K-slabs in
// fragment order (m0 a multiple of 16).  SKIP: waves with pos.active == false only move operands.
template <bool WARM, bool SWAP, bool BT = false, bool AF = false, bool SKIP = false>
__device__ __forceinline__ void gemm_tile_dma(const DmaOperand& A, const DmaOperand& B, int K, int m0, int n0,
                                              const WavePos& pos, uint16_t* smem, Acc& acc) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int wm = pos.wm, wn = pos.wn;
  acc_zero(acc);
  const int nk = K / kDK;
  if (nk == 0) return;
  const __amdgpu_buffer_rsrc_t ra = operand_rsrc(A), rb = operand_rsrc(B);
  static_assert(!(WARM && BT), "the warm-up assumes K-contiguous operands");
  const DmaLane la = AF ? dma_lane_af(m0, A, wave, lane) : dma_lane(m0, A, wave, lane);
  const DmaLane lb = BT ? dma_lane_bt(n0, B.ld, wave, lane) : dma_lane(n0, B, wave, lane);
  auto load_b = [&](Frags& f, const uint16_t* Bs, int ks) {
    if constexpr (BT) frags_load_bt(f, Bs, wn * 64, ks, lane);
    else frags_load(f, Bs, wn * 64, ks, lane);
  };
  auto load_a = [&](Frags& f, const uint16_t* As, int half, int ks) {
    if constexpr (AF) {
#pragma unroll
      for (int i = 0; i < kFragBlocks; ++i)
        f[i] = *reinterpret_cast<const bf16x8_t*>(As + (wm * 8 + half * kFragBlocks + i) * 1024 + ks * 512 + lane * 8);
    } else {
      frags_load(f, As, wm * 128 + half * 64, ks, lane);
    }
  };
  dma_issue(ra, rb, la, lb, 0, smem, wave);
  // L2 warm-up.  A fifth of a slice's lines miss L2 (the 32 workgroups resident on an XCD form an
  // 8 x 4 block of tiles: 12 operand slices for 32 tiles), and loads return in order, so one late
  // line holds back everything queued behind it.  Each slice is therefore touched two slices
  // early with one 4-byte load per 128-byte line (sunk into a scratch corner of LDS), the lines
  // shared out over the workgroups that will read them: wave 0 takes a quarter of the A rows
  // (which quarter: by tile column), wave 4 an eighth of the B rows (by tile row).  The touch is
  // issued late in the slice, when every wave's requests for the next slice are already queued
  // ahead of it, and it may stay in flight across the next barrier (vmcnt(1)).
  constexpr int kWarmAhead = 2;
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);   // wave-uniform: the descriptor stays scalar
  const bool warm_a = wave_u < 4, warm_wave = WARM && (wave_u & 3) == 0;
  const __amdgpu_buffer_rsrc_t rw = warm_a ? ra : rb;
  const int warm_row = warm_a ? m0 + ((n0 / kTile) & 3) * 64 + lane : n0 + ((m0 / kTile) & 7) * 32 + (lane & 31);
  const uint32_t warm_off = uint32_t(int64_t(warm_row) * (warm_a ? A.ld : B.ld) * 2) + (warm_a ? 0u : uint32_t(lane >> 5) * 64u);
  const uint32_t warm_kstep = uint32_t((warm_a ? A.kstep : B.kstep) * 2);
  uint16_t* const warm_sink = smem + kWarmSinkOff / 2 + wave * 128;
  if constexpr (SKIP) {
    if (!pos.active) {   // uniform over the wave: its part of the transfers, the same barriers, no arithmetic
      for (int kt = 0; kt < nk; ++kt) {
        __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
        AERO_CFENCE();
        __builtin_amdgcn_s_barrier();
        AERO_CFENCE();
        if (kt + 1 < nk) dma_issue(ra, rb, la, lb, kt + 1, smem + ((kt + 1) & 1) * kDStageElems, wave);
      }
      __syncthreads();
      return;
    }
  }
  // One iteration = one 64-wide slice = two 32-wide K steps of two halves, 16 MFMAs per wave each.
  // The order is pinned with scheduling barriers: the first step's fragments are read up front, the
  // next slice is requested only after the first MFMA group (issuing the 8 loads right after the
  // barrier would hold back every wave's first MFMAs: measured 8 % slower), and the other fragment
  // reads are interleaved with MFMAs, two per read.
  // warm: touch slice kt + kWarmAhead; warm_pending: the previous slice issued a touch.
  auto slice = [&](int kt, bool prefetch, bool warm, bool warm_pending) {
    // slice kt landed (the youngest load may be a touch: loads return in order), own LDS reads done
    if (warm_pending && warm_wave) __builtin_amdgcn_s_waitcnt(0x0071);   // vmcnt(1) lgkmcnt(0)
    else __builtin_amdgcn_s_waitcnt(0x0070);                             // vmcnt(0) lgkmcnt(0)
    AERO_CFENCE();
    __builtin_amdgcn_s_barrier();
    AERO_CFENCE();
    const uint16_t* As = smem + (kt & 1) * kDStageElems;
    const uint16_t* Bs = As + kTile * kDK;
    Frags b0, b1, a0, a1, a2;
    load_a(a0, As, 0, 0);
    load_b(b0, Bs, 0);
    load_a(a1, As, 1, 0);
    frags_mma<SWAP>(a0, b0, 0, acc);
    if (prefetch) dma_issue(ra, rb, la, lb, kt + 1, smem + ((kt + 1) & 1) * kDStageElems, wave);
    load_a(a2, As, 0, 1);
    load_b(b1, Bs, 1);
    frags_mma<SWAP>(a1, b0, 1, acc);
    load_a(a0, As, 1, 1);
    frags_mma<SWAP>(a2, b1, 0, acc);
    constexpr int kMfma = 0x008, kVmemRd = 0x020, kDsRd = 0x100;
    constexpr int kMfmas = kFragBlocks * kNB;
    constexpr int kReadsB = BT ? 2 * kFragBlocks : kFragBlocks;
    __builtin_amdgcn_sched_group_barrier(kDsRd, 2 * kFragBlocks + kReadsB, 0);
    __builtin_amdgcn_sched_group_barrier(kMfma, kMfmas, 0);
    if (prefetch) __builtin_amdgcn_sched_group_barrier(kVmemRd, 8, 0);
#pragma unroll
    for (int r = 0; r < kFragBlocks; ++r) {
      __builtin_amdgcn_sched_group_barrier(kMfma, 2, 0);
      __builtin_amdgcn_sched_group_barrier(kDsRd, 1, 0);
      __builtin_amdgcn_sched_group_barrier(kMfma, 2, 0);
      __builtin_amdgcn_sched_group_barrier(kDsRd, kReadsB / kFragBlocks, 0);
    }
#pragma unroll
    for (int r = 0; r < kFragBlocks; ++r) {
      __builtin_amdgcn_sched_group_barrier(kMfma, 2, 0);
      __builtin_amdgcn_sched_group_barrier(kDsRd, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(kMfma, 2 * kMfmas - 6 * kFragBlocks, 0);
    if (WARM) {
      __builtin_amdgcn_sched_barrier(0);
      if (warm && warm_wave)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, warm_sink, 4, warm_off + uint32_t(kt + kWarmAhead) * warm_kstep, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    frags_mma<SWAP>(a0, b1, 1, acc);
    if (!WARM) __builtin_amdgcn_sched_group_barrier(kMfma, kMfmas, 0);
  };
  // Every call site passes constants, so that each copy of the slice is one scheduling region.
  // Measured: worth 2-4 % per contraction from about 50 slices on, nothing or a small loss at 24.
  constexpr int kWarmMinSlices = 32;
  if (WARM && nk >= kWarmMinSlices) {   // slice kt touches slice kt + 2: all but the last two do
    slice(0, true, true, false);
    for (int kt = 1; kt + kWarmAhead < nk; ++kt) slice(kt, true, true, true);
    slice(nk - 2, true, false, true);
    slice(nk - 1, false, false, false);
  } else {
    for (int kt = 0; kt + 1 < nk; ++kt) slice(kt, true, false, false);
    slice(nk - 1, false, false, false);
  }
  __syncthreads();
}

// Picks the fast loop when its preconditions hold (uniform over the launch).
__device__ __forceinline__ void gemm_tile_auto(const uint16_t* __restrict__ A, int64_t lda, int M,
                                               const uint16_t* __restrict__ B, int64_t ldb, int N, int K,
                                               int m0, int n0, const WavePos& pos, uint16_t* smem, Acc& acc) {
  const bool fast = (K % kDK == 0) && (lda % 8 == 0) && (ldb % 8 == 0) &&
                    (reinterpret_cast<uintptr_t>(A) % 16 == 0) && (reinterpret_cast<uintptr_t>(B) % 16 == 0) &&
                    ((int64_t(M) - 1) * lda + K) < (int64_t(1) << 31) && ((int64_t(N) - 1) * ldb + K) < (int64_t(1) << 31);
  if (fast) gemm_tile_dma<true, false, false, false, true>(operand_row_major(A, lda, M, K), operand_row_major(B, ldb, N, K), K, m0,
                                                           n0, pos, smem, acc);
  else gemm_tile<false>(A, lda, M, B, ldb, N, K, m0, n0, pos, smem, acc);
}

}  // namespace aero
