// bf16 MFMA GEMM tile for gfx950: D[256 x 256] (fp32) = A[256 x K] * B[256 x K]^T, both
// operands row-major with K contiguous.  One workgroup of 8 waves (2 x 4, two per SIMD) owns
// the tile; each wave accumulates a 128 x 64 sub-tile as 8 x 4 blocks of
// v_mfma_f32_16x16x32_bf16.  Two waves per SIMD let one wave's waits (barrier, LDS latency,
// epilogue arithmetic) hide behind the other's matrix instructions.
//
// Two things bound the loop, in about equal parts.  The power limit: k_fused_stats<false> at 151936 x 16384 x 1536 takes
// 5.74 ms on Gaussian operands at 1.85 GHz and 4.54 on zeros at 2.39, the matrix units busy in 66-69 % of the cycles both
// times, so the energy per flop of the matrix instruction counts; a stream of nothing but 16 x 16 x 32 reaches 2.11
// PFLOP/s on Gaussian data where 32 x 32 x 16 reaches 1.85 (both 2.4-2.5 on zeros), and 2.13 when consecutive
// instructions always share one operand (the column order alternates from row to row).  And the other third of the
// cycles, part of which the clock would take back: the library's 81 % at K = 3584 come with 1.73 GHz.  The bare loop below:
// 1.45 PFLOP/s at 151936 x 16384 x 1536 and 1.44 at 152064 x 32768 x 3584, against 1.36 / 1.34 with 32 x 32 x 16.
//
// Operands go HBM -> LDS directly (buffer_load ... lds) in two stages of 256 x 64 slices; rows start on 16 bytes, K is any
// multiple of 8.  (A loop that staged slices through registers took the rows whose length is no multiple of 64: forward of
// 2500 tokens at H = 600, V = 32000 220 us, 130 this way.)
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
constexpr size_t kEpilogueOff = kWarmSinkOff + 2048;   // + a 256-byte sink per wave for the warm-up loads
constexpr size_t kGemmLdsBytes = kEpilogueOff + 5120;   // + what an epilogue uses: the stages hold the next tile's slices

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

// Lines of an operand's slice (256) that a tile touches for all that share them: wave `turn` of four takes the first 64.
struct WarmShare {
  int first, last, turn;
};

// Which part of the tile a wave owns.  Waves w and w + 4 run on the same SIMD; the two that share one are the halves
// of the dimension that may be ragged, so that skipping waves whose rows or columns are all padding halves the work
// of every SIMD: rows of A (wave_pos<false>) or columns of B, in steps of two blocks of 64 (wave_pos<true>).
// Whole calls at H = 1536, V = 151936: 600 tokens (a third tile with 88) 905 -> 873 us, 1100 and 16384 tokens even;
// 1400 tokens at H = 3584, V = 32000 826 -> 815; 300 tokens at H = 896, V = 8000 102.2 -> 103.7.
struct WavePos {
  int wm, wn;
  bool active;                // false: all of the wave's rows (columns) are padding, its accumulators stay zero
  WarmShare warm_a, warm_b;   // this tile's share of the L2 warm-up
  int warm_from;              // it is done for tiles of at least this many slices
};
// From how many slices on.
//   dweight     from 32: worth 2-4 % from about 50 slices on, from 8 on it cost 0-1.5 % up to 6000 tokens.
//   forward     from 12, with one token tile from 8: the weight comes from memory once per band of tiles, and a workgroup that walks its
//               tiles waits for a late line itself.  Forward-only calls without / with it, the weight not in the memory-side cache (other
//               work came between) and, in brackets, left there by the call before: H = 1536, V = 151936 500 tokens 286 / 249 us (251 / 221),
//               700 340 / 331 (316 / 321), 900 455 / 385 (418 / 391), 1700 695 / 675 (680 / 676), 3300 1288 / 1219 (1255 / 1217); H = 1024 500
//               tokens 202 / 171 (169 / 156), 700 233 / 234 (206 / 206), 1400 398 / 374 (386 / 384); H = 768 500 tokens 174 / 143 (120 / 121), 700
//               200 / 192 (156 / 158), 900 265 / 225 (204 / 210), 1700 366 / 359 (347 / 349), 3300 656 / 643 (639 / 640); with a gradient 0.94-1.02
//               of the time without.
//   dhidden     not at all: its loop requests further ahead (GemmRing), and has more than one touch of a line to lose by it.
constexpr int kWarmSlices = 32, kWarmSlicesForward = 12, kWarmSlicesAlone = 8;
__device__ __forceinline__ int forward_warm_from(int token_tiles) {
  return token_tiles == 1 ? kWarmSlicesAlone : kWarmSlicesForward;
}
// The lines in equal parts to the tiles that have the slice in common, a quarter where there are four or more.  (Three tiles with
// whole quarters, two of them twice: 768 tokens at H = 3584 815 us forward, 724 this way.)
__device__ __forceinline__ WarmShare warm_share(int index, int sharers) {
  const int parts = min(max(sharers, 1), 4), part = index % parts;
  const int lines = (kTile + parts - 1) / parts;
  return WarmShare{part * lines, min((part + 1) * lines, kTile) - 1, part};
}
template <bool RAGGED_COLS> __device__ __forceinline__ WavePos wave_pos() {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  return RAGGED_COLS ? WavePos{wave & 1, wave >> 1, true, {}, {}, 0} : WavePos{wave >> 2, wave & 3, true, {}, {}, 0};
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

// The tile that a workgroup of a walking grid (a multiple of 8 workgroups, so that a walk stays on its XCD) has at
// step pid = blockIdx.x, + gridDim.x, ...  tile0: position in the tile order of the launch's first tile, n: its tiles (a
// kernel's tiles may be spread over several launches).  False: none, the walk has ended.
__device__ __forceinline__ bool tile_of_step(int pid, int tiles_m, int tiles_n, int tile0, int n, int& tm, int& tn) {
  const int pos = xcd_position(pid, n);
  tile_of_index(tile0 + max(pos, 0), tiles_m, max(tiles_n, 1), tm, tn);
  return pos >= 0;
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

constexpr int kDK = 64;                          // K slice of the loop
constexpr int kDStageElems = 2 * kTile * kDK;    // A then B
static_assert(size_t(2) * kDStageElems * 2 <= kGemmStageBytes, "two stages must fit the LDS budget");

// Rows are 128 bytes; rows of equal parity share a 128-byte half of the 256-byte bank line, so
// the chunk index is swizzled with bits 1..3 of the row: 16 consecutive rows -> 16 distinct slots.
__device__ __forceinline__ int lds_off(int row, int chunk) {
  return row * kDK + ((chunk ^ ((row >> 1) & 7)) << 3);
}

// Where a lane finds its fragments in an operand's slice, as LDS byte addresses: `at` per K step or per block, whichever
// the layout's swizzle makes differ, everything else in the instructions' offsets.  They are kept in registers from slice
// to slice (formed behind the barrier they cost the first reads 1 % of the dhidden contraction).
typedef __attribute__((address_space(3))) uint16_t lds_u16_t;
__device__ __forceinline__ uint32_t lds_address(const uint16_t* p) { return uint32_t(uintptr_t((lds_u16_t*)p)); }
__device__ __forceinline__ bf16x8_t lds_fragment(uint32_t address) {
  typedef __attribute__((address_space(3))) const bf16x8_t lds_frag_t;
  return *(lds_frag_t*)uintptr_t(address);
}
template <int N> struct FragAddr {
  uint32_t at[N];
  __device__ __forceinline__ void move(uint32_t by) {
#pragma unroll
    for (int k = 0; k < N; ++k) {
      at[k] += by;
      asm volatile("" : "+v"(at[k]));
    }
  }
};
// K-contiguous rows, swizzled: at[ks] is K step ks of row row0; block i lies 16 rows behind.
__device__ __forceinline__ FragAddr<2> frag_addr(const uint16_t* lds, int row0, int lane) {
  const int row = row0 + (lane & 15), g = lane >> 4;
  return FragAddr<2>{{lds_address(lds) + lds_off(row, g) * 2, lds_address(lds) + lds_off(row, 4 + g) * 2}};
}
__device__ __forceinline__ void frags_load(Frags& f, const FragAddr<2>& from, int first, int ks) {
#pragma unroll
  for (int i = 0; i < kFragBlocks; ++i) f[i] = lds_fragment(from.at[ks] + (first + i) * 16 * kDK * 2);
}
// Fragment order: blocks of 2 KB, the two K steps one after the other.
__device__ __forceinline__ FragAddr<1> frag_addr_af(const uint16_t* lds, int row0, int lane) {
  return FragAddr<1>{{lds_address(lds) + row0 * kDK * 2 + lane * 16}};
}
__device__ __forceinline__ void frags_load(Frags& f, const FragAddr<1>& from, int first, int ks) {
#pragma unroll
  for (int i = 0; i < kFragBlocks; ++i) f[i] = lds_fragment(from.at[0] + (first + i) * 2048 + ks * 1024);
}

// ------------------------------------------------------------------------------------------
// Direct-to-LDS loop.  buffer_load ... lds moves 16 bytes per lane from HBM/L2 straight into
// LDS (lane l of a wave lands at LDS base + 16 l): no staging registers, no LDS stores, and the
// buffer descriptor's bounds check turns rows past the operand's end into zeros.  Slices are
// 256 x 64: every row contributes one full 128-byte line per slice (32-wide slices fetch half
// lines and lose a tenth of the throughput), two stages of 64 KB.
//
// Completion of these loads is tracked by hand: vmcnt(0) in front of the barrier means this
// wave's part of the slice has landed, the barrier then makes every wave's part visible and
// also guarantees that the other stage is no longer being read.  The compiler does not model
// these dependencies, hence the explicit waits and compiler fences.
// ------------------------------------------------------------------------------------------
// An operand: rows of 64-wide K slices.  Element (row, k) lives at
//   base + (k / 64) * kstep + row * ld + k % 64
//   row-major [rows, K]:            ld = row pitch, kstep = 64
//   K-slabs [rows/256][K/64][256][64]: ld = 64, kstep = 256 * 64: the layout of the library's own intermediate operands.
//       A slice is one 32 KB block and a tile's slices follow each other, so that a workgroup reads one contiguous run
//       and the forward contraction writes 128 KB pieces.  (As [K/64][rows][64], a slab of 2-8 MB for every 64 of K and so a new
//       page with every slice: dweight 1608 / 1539 us for 1536 tiles of 167 slices and 3906 / 3745 for 1792 of 333, the
//       forward contraction with its stores 0 to 1.5 %.)
// and loads past its bytes return zeros.
// K-slabs in fragment order (AF): inside a slab every 16 rows are one 2 KB block, the two 32-wide K steps one after
// the other, each as the 16 x 16 x 32 instruction's lanes hold it.  A wave's accumulators can be stored in it straight
// from registers, 1 KB per instruction, and a fragment is 1 KB of LDS read lane by lane.
constexpr int kSlabElems = kTile * 64;
__device__ __forceinline__ int64_t slab_offset(int64_t slabs, int64_t tile, int64_t slab) { return (tile * slabs + slab) * kSlabElems; }
__device__ __forceinline__ int64_t frag_order_offset(int64_t slabs, int64_t row, int64_t k) {
  return slab_offset(slabs, row / kTile, k / 64) + (row % kTile / 16) * 1024 + (k % 64 / 32) * 512 + (k % 32 / 8) * 128 + (row % 16) * 8 + k % 8;
}
__device__ __forceinline__ __amdgpu_buffer_rsrc_t operand_rsrc(const uint16_t* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), 0, int(bytes), 0x00020000);
}

#define AERO_CFENCE() asm volatile("" ::: "memory")

// Per-lane byte offsets of the DMA loads of one operand, from the tile's first row on.  Wave w fills rows
// [32 w, 32 w + 32) with 4 instructions of 8 rows; lane l covers row l/8 of those 8 and LDS slot l%8, and the
// chunk that belongs in that slot is slot ^ ((row >> 1) & 7) with row = 32 w + 8 j + l/8, i.e.
// (l % 8) ^ ((4 j + l / 16) & 7): one offset for even j, one for odd j.
struct DmaLane {
  uint32_t even, odd, row_step, k_step;
};
__device__ __forceinline__ uint32_t dma_chunk(int lane, int j) { return uint32_t((lane & 7) ^ ((4 * j + (lane >> 4)) & 7)); }
__device__ __forceinline__ DmaLane dma_lane(int64_t ld, int64_t kstep, int wave, int lane) {
  const uint32_t row = uint32_t(int64_t(wave * 32 + (lane >> 3)) * ld * 2);
  return DmaLane{row + dma_chunk(lane, 0) * 16, row + dma_chunk(lane, 1) * 16, uint32_t(8 * ld * 2), uint32_t(kstep * 2)};
}

// The same for an operand in fragment order: a wave's 32 rows are 4 KB in one piece.
__device__ __forceinline__ DmaLane dma_lane_af(int64_t kstep, int wave, int lane) {
  const uint32_t at = uint32_t(wave * 32 * kDK * 2 + lane * 16);
  return DmaLane{at, at, 1024u, uint32_t(kstep * 2)};
}

// An operand stored the other way round (BT): a row-major matrix whose rows are the contraction index, [K][rows],
// e.g. the weight in dhidden = dz weight (GemmRing).  A step is 32 rows of 256 columns (512 bytes, whole lines); its LDS
// image keeps that orientation, [32][256], and fragments come out of it with the transposing LDS read
// (ds_read_b64_tr_b16): of every 16 lanes, lane j names four consecutive columns 4 (j % 4) .. of row j / 4, and
// receives column j of those four rows, so two reads make the eight K values of a fragment.  The 32-byte
// segments of a row are XORed with f(row) = row % 4 + 4 ((row / 8) % 2): the eight rows that 32 lanes touch at once
// fall on distinct banks.
__device__ __forceinline__ FragAddr<4> frag_addr_bt(const uint16_t* lds, int col0, int lane) {
  const int group = lane >> 4, j = lane & 15;
  const int swz = (j >> 2) | (group & 1) << 2;
  FragAddr<4> a;
#pragma unroll
  for (int i = 0; i < kFragBlocks; ++i)
    a.at[i] = lds_address(lds) + ((group * 8 + (j >> 2)) * kTile + (j & 3) * 4 + ((col0 / 16 + i) ^ swz) * 16) * 2;
  return a;
}
__device__ __forceinline__ void frags_load(Frags& f, const FragAddr<4>& from, int, int ks) {
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  typedef short s16x8_t __attribute__((ext_vector_type(8)));
  typedef __attribute__((address_space(3))) s16x4_t lds_s16x4_t;
#pragma unroll
  for (int i = 0; i < kFragBlocks; ++i) {
    const uint32_t at = from.at[i] + ks * 32 * kTile * 2;
    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)uintptr_t(at));
    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_t*)uintptr_t(at + 4 * kTile * 2));
    const s16x8_t both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    f[i] = __builtin_bit_cast(bf16x8_t, both);
  }
}

__device__ __forceinline__ void slice_barrier() {
  AERO_CFENCE();
  __builtin_amdgcn_s_barrier();
  AERO_CFENCE();
}
// Barrier of an epilogue that exchanges through LDS: waits for the wave's own LDS accesses, not for the next tile's
// operands on their way, as __syncthreads would.
__device__ __forceinline__ void lds_barrier() {
  AERO_CFENCE();
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  slice_barrier();
}
// A copy that the compiler does not see through: what an epilogue derives from it is formed per tile, not kept in
// registers beside the main loop's.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}
// Nothing that a wave has requested into LDS is on its way when it leaves.
__device__ __forceinline__ void end_of_walk() {
  AERO_CFENCE();
  __builtin_amdgcn_s_waitcnt(0x0070);
}

// One tile's operands: where its K range starts in each (a: bytes from a_base to row m0's first slice, likewise b), the
// bytes that bound them, and how many slices there are.
struct TileSrc {
  const uint16_t *a_base, *b_base;
  int64_t a_bytes, b_bytes;
  uint32_t a, b;
  int nk;
};

// What follows a workgroup's last tile: no bytes, so that requesting it moves nothing.
__device__ __forceinline__ TileSrc no_tile(const TileSrc& t) { return TileSrc{t.a_base, t.b_base, 0, 0, 0u, 0u, 1}; }

// The main loop of a workgroup that walks tiles.  Slices form one stream across tiles: every slice requests the next one,
// and a tile's last slice the next tile's first, so that a tile's epilogue runs while its successor's operands are on
// their way.  A workgroup per tile lost between 3 and 8 us a tile to the launch, the first slice's latency and
// the drain of the stores, of 45 us at 24 slices and 17 at 7.  Tile by tile / walking: k_fused_stats<true> with 16384 tokens at
// H = 1536, V = 151936 6.72 / 6.44 ms, at H = 3584 13.88 / 13.77, 1200 tokens 614 / 595 us; k_gemm_dw 600 tokens 229 / 215 us; from
// about 100 slices on a workgroup per tile is the faster way there (kDwTileRows), by launching one.  Tried on top and not taken: starts staggered over the CUs (0 to +20 %: tiles
// do not wait for each other's stores), waves 4 to 7 free of loads and warming L2 four slices ahead (dweight of 1000
// tokens -8 %, everything long +3 to +12 %: bytes into the CU are what counts).
// WARM: L2 warm-up two slices ahead (see kWarmSlices).
// AF: operand A is in K-slabs in fragment order (tiles start at multiples of 16 rows).
// TAIL: K need not be a multiple of 64: the 16-byte chunks of the last slice that lie past a row's end are requested from
// behind the buffer, which gives zeros.
template <bool WARM, bool SWAP, bool AF, bool TAIL>
struct GemmStream {
  DmaLane la, lb;
  int lane, wave, stage;   // stage: where the next slice lies
  int tail;                // 16-byte chunks of a row's last slice

  // lda, ldb: row pitches; kstep_a, kstep_b: elements between slices; K: the row length with TAIL
  __device__ __forceinline__ GemmStream(int64_t lda, int64_t kstep_a, int64_t ldb, int64_t kstep_b, int K) {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    stage = 0;
    la = AF ? dma_lane_af(kstep_a, wave, lane) : dma_lane(lda, kstep_a, wave, lane);
    lb = dma_lane(ldb, kstep_b, wave, lane);
    tail = TAIL ? (K - 1) % kDK / 8 + 1 : 8;
  }

  // Requests slice kt of a tile into a stage; LAST: it may be the tile's last one.  The whole byte offset travels in the vector offset: the hardware bounds
  // check covers the vector offset only, not the scalar one.
  template <bool LAST>
  __device__ __forceinline__ void issue(const TileSrc& t, int kt, uint16_t* to) {
    const __amdgpu_buffer_rsrc_t ra = operand_rsrc(t.a_base, t.a_bytes), rb = operand_rsrc(t.b_base, t.b_bytes);
    uint16_t* a_dst = to + wave * 32 * kDK;
    uint16_t* b_dst = to + kTile * kDK + wave * 32 * kDK;
    const uint32_t a = t.a + uint32_t(kt) * la.k_step, b = t.b + uint32_t(kt) * lb.k_step;
    uint32_t past_even = 0, past_odd = 0;   // all ones (but 16) where the lane's chunk does not exist
    if constexpr (TAIL && LAST) {
      const int l = opaque(lane), chunks = kt + 1 == t.nk ? tail : 8;
      past_even = int(dma_chunk(l, 0)) >= chunks ? ~15u : 0u;
      past_odd = int(dma_chunk(l, 1)) >= chunks ? ~15u : 0u;
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      uint32_t oa = ((j & 1) ? la.odd : la.even) + (a + j * la.row_step), ob = ((j & 1) ? lb.odd : lb.even) + (b + j * lb.row_step);
      if constexpr (TAIL && LAST) {
        oa |= (j & 1) ? past_odd : past_even;
        ob |= (j & 1) ? past_odd : past_even;
      }
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, a_dst + j * 8 * kDK, 16, oa, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, b_dst + j * 8 * kDK, 16, ob, 0, 0, 0);
    }
  }

  __device__ __forceinline__ void start(const TileSrc& t, uint16_t* smem) { issue<true>(t, 0, smem + stage * kDStageElems); }

  // acc = the tile's product.  Its first slice has been requested; on return the first one of `next` has (one of no bytes,
  // which moves nothing, if the walk ends here).  PENDING: how many memory operations every wave is sure to have issued
  // since then, in program order, if `stores` (they need not have completed).
  // active == false: all of the wave's rows (columns) are padding, it only moves operands.
  template <int PENDING>
  __device__ __forceinline__ void run(const TileSrc& t, const TileSrc& next, const WavePos& pos, bool stores, uint16_t* smem, Acc& acc) {
    const int wm = pos.wm, wn = pos.wn, nk = t.nk;
    acc_zero(acc);
    // the first slice has landed: requested before the epilogue's stores
    if (stores) __builtin_amdgcn_s_waitcnt(0x0070 | (PENDING & 15) | (PENDING >> 4) << 14);
    else __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0) lgkmcnt(0)
    slice_barrier();
    if (!pos.active) {   // uniform over the wave: its part of the transfers, the same barriers, no arithmetic
      for (int kt = 0; kt + 1 < nk; ++kt) {
        issue<true>(t, kt + 1, smem + (stage ^ 1) * kDStageElems);
        stage ^= 1;
        __builtin_amdgcn_s_waitcnt(0x0070);
        slice_barrier();
      }
      issue<true>(next, 0, smem + (stage ^ 1) * kDStageElems);
      stage ^= 1;
      return;
    }
    // L2 warm-up.  A fifth of a slice's lines miss L2 (the 32 workgroups resident on an XCD form an
    // 8 x 4 block of tiles: 12 operand slices for 32 tiles), and loads return in order, so one late
    // line holds back everything queued behind it.  Each slice is therefore touched two slices
    // early with one 4-byte load per 128-byte line (sunk into a scratch corner of LDS), the lines
    // shared out over the workgroups that will read them (warm_share): waves 0 to 3 take the A rows' lines, 4 to 7 those of B.  The touch is issued late in the slice, when every wave's
    // requests for the next slice are already queued ahead of it, and it may stay in flight across the next barrier
    // (vmcnt(1)).
    constexpr int kWarmAhead = 2;
    const bool warm_a = wave < 4;
    const WarmShare& warm = warm_a ? pos.warm_a : pos.warm_b;
    const int warm_at = warm.first + ((wave - warm.turn) & 3) * 64;
    const bool warm_wave = warm_at <= warm.last;
    const __amdgpu_buffer_rsrc_t rw = warm_a ? operand_rsrc(t.a_base, t.a_bytes) : operand_rsrc(t.b_base, t.b_bytes);
    const uint32_t line = uint32_t(min(warm_at + lane, warm.last));
    const uint32_t warm_off = warm_a ? t.a + line * (la.row_step / 8) : t.b + line * (lb.row_step / 8);
    const uint32_t warm_kstep = warm_a ? la.k_step : lb.k_step;
    uint16_t* const warm_sink = smem + kWarmSinkOff / 2 + wave * 128;
    const uint16_t* const first = smem + stage * kDStageElems;
    auto fa = [&] {
      if constexpr (AF) return frag_addr_af(first, wm * 128, lane);
      else return frag_addr(first, wm * 128, lane);
    }();
    auto fb = frag_addr(first + kTile * kDK, wn * 64, lane);
    // One iteration = one 64-wide slice = two 32-wide K steps of two halves, 16 MFMAs per wave each.
    // The order is pinned with scheduling barriers: the first step's fragments are read up front, the
    // next slice is requested only after the first MFMA group (issuing the 8 loads right after the
    // barrier would hold back every wave's first MFMAs: measured 8 % slower), and the other fragment
    // reads are interleaved with MFMAs, two per read.
    // (src, kn): the slice after this one; touch: the one that is touched.
    auto slice = [&](auto last, auto touching, const TileSrc& src, int kn, int touch) {
      Frags b0, b1, a0, a1, a2;
      constexpr int kMfma = 0x008, kVmemRd = 0x020, kDsRd = 0x100;
      constexpr int kMfmas = kFragBlocks * kNB;
      frags_load(a0, fa, 0, 0);
      frags_load(b0, fb, 0, 0);
      __builtin_amdgcn_sched_barrier(0);   // these first: the matrix instructions start with them
      frags_load(a1, fa, kFragBlocks, 0);
      frags_mma<SWAP>(a0, b0, 0, acc);
      issue<decltype(last)::value>(src, kn, smem + (stage ^ 1) * kDStageElems);
      frags_load(a2, fa, 0, 1);
      frags_load(b1, fb, 0, 1);
      frags_mma<SWAP>(a1, b0, 1, acc);
      frags_load(a0, fa, kFragBlocks, 1);
      frags_mma<SWAP>(a2, b1, 0, acc);
      __builtin_amdgcn_sched_group_barrier(kDsRd, kFragBlocks, 0);
      __builtin_amdgcn_sched_group_barrier(kMfma, kMfmas, 0);
      __builtin_amdgcn_sched_group_barrier(kVmemRd, 8, 0);
#pragma unroll
      for (int r = 0; r < 2 * kFragBlocks; ++r) {
        __builtin_amdgcn_sched_group_barrier(kMfma, 2, 0);
        __builtin_amdgcn_sched_group_barrier(kDsRd, 1, 0);
      }
#pragma unroll
      for (int r = 0; r < kFragBlocks; ++r) {
        __builtin_amdgcn_sched_group_barrier(kMfma, 2, 0);
        __builtin_amdgcn_sched_group_barrier(kDsRd, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(kMfma, 2 * kMfmas - 6 * kFragBlocks, 0);
      constexpr bool kTouch = decltype(touching)::value;
      if constexpr (kTouch) {
        __builtin_amdgcn_sched_barrier(0);
        if (warm_wave)
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, warm_sink, 4, warm_off + uint32_t(touch) * warm_kstep, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      frags_mma<SWAP>(a0, b1, 1, acc);
      if constexpr (!kTouch) __builtin_amdgcn_sched_group_barrier(kMfma, kMfmas, 0);
      stage ^= 1;
      __builtin_amdgcn_sched_barrier(0);   // what follows stays behind the last matrix instruction
    };
    auto landed = [&](auto touched) {   // the next slice (the youngest load may be a touch: loads return in order), own LDS reads done
      const uint32_t by = stage ? uint32_t(kDStageElems * 2) : 0u - uint32_t(kDStageElems * 2);   // stage: that slice's
      fa.move(by);
      fb.move(by);
      if (decltype(touched)::value && warm_wave) __builtin_amdgcn_s_waitcnt(0x0071);   // vmcnt(1) lgkmcnt(0)
      else __builtin_amdgcn_s_waitcnt(0x0070);
      slice_barrier();
    };
    constexpr std::false_type kNo{};
    constexpr std::true_type kYes{};
    constexpr int kPeel = TAIL ? 2 : 1;
    // A scalar load on its way into the loop (an argument that only the epilogue needs) would make the compiler wait for
    // every fragment before the first matrix instruction of each slice.
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
    int kt = 0;
    if constexpr (WARM) {
      if (nk >= pos.warm_from)
        for (; kt + kWarmAhead < nk; ++kt) {
          slice(kNo, kYes, t, kt + 1, kt + kWarmAhead);
          landed(kYes);
        }
    }
    for (; kt + kPeel < nk; ++kt) {
      slice(kNo, kNo, t, kt + 1, 0);
      landed(kNo);
    }
    if (TAIL && kt + 1 < nk) {
      slice(kYes, kNo, t, kt + 1, 0);
      landed(kNo);
    }
    slice(kYes, kNo, next, 0, 0);
  }
};

// ------------------------------------------------------------------------------------------
// Ring loop: A in K-slabs in fragment order, B stored the other way round ([K][rows], see above), operands of the matrix
// instruction exchanged; one tile per workgroup.
//
// A stage of the loop above is requested one slice ahead, and with a transposed operand only behind all of that slice's
// transposing reads, which the compiler holds back for every load into LDS that it knows of.  Here a stage is one 32-wide K
// step (both layouts keep whole lines: 1 KB blocks of A, 512-byte rows of B), four of them lie in LDS, and a step is requested
// three steps before it is read, in instructions that the compiler does not count.  The second half of a step's matrix
// instructions waits until the barrier behind it, and covers the reads of the next step's first fragments.
// k_gemm_dh, two stages of 64 / this loop: 600 tokens at H = 1536, V = 151936 with 390 candidates 208 / 184 us, with 600 296 / 267, 16384 with
// 5/8 of them candidates 4047 / 3635, 32768 at H = 3584, V = 152064 with 65 % 20.15 / 18.08 ms.  Where the requests stand: in front of the first group of matrix instructions 3781 and 19033 against
// 3635 and 18085; one every four instructions and by half of the waves no better, the latter 4200.
// (For dweight, whose operands are both in fragment order, 1612 / 1539: it keeps the loop above.)
// ------------------------------------------------------------------------------------------
constexpr int kStepK = 32, kRing = 4;
constexpr int kStepBytes = 2 * kTile * kStepK * 2;   // A, then B
static_assert(size_t(kRing) * kStepBytes <= kGemmStageBytes, "the ring must fit the LDS budget");

typedef uint32_t rsrc_words_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ rsrc_words_t rsrc_words(const uint16_t* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  return rsrc_words_t{uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(b))), uint32_t(__builtin_amdgcn_readfirstlane(uint32_t(b >> 32))) & 0xffffu,
                      uint32_t(__builtin_amdgcn_readfirstlane(bytes)), 0x00020000u};
}
// buffer_load_dwordx4 ... lds: 16 bytes a lane, to LDS byte address `to` (uniform, in M0) + 16 lane.  It has no destination register
// that the compiler could take for written; the loop waits for it by vmcnt.  What the compiler does not know of it:
//   M0, which its own loads into LDS use as well, is written: declared, as an output, since it takes no clobber of it.  (As an
//     input that the compiler puts there, the calls of 16384 tokens and more were 0.6 % slower.)
//   LDS is written, later.  That is not declared (a "memory" clobber would hold back the step's reads of other stages): a stage is never
//     read and requested between the same two calls of landed, whose wait, barrier and fence order the ones behind the others.
//   A scalar register that a vector instruction wrote (v_readfirstlane) may be read by a load only five wait states later: the
//     descriptors are formed once, in front of the loop, and the wait states follow them there (descriptors_settled).
__device__ __forceinline__ void request_lds16(rsrc_words_t r, uint32_t to, uint32_t off) {
  uint32_t m0;
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %2, %3, 0 offen lds" : "=&{m0}"(m0) : "s"(to), "v"(off), "s"(r));
}
__device__ __forceinline__ void descriptors_settled(rsrc_words_t a, rsrc_words_t b) { asm volatile("s_nop 4" ::"s"(a), "s"(b)); }

struct RingSrc {
  const uint16_t *a_base, *b_base;   // the K range's first slab of the tile, the first K row
  uint32_t a_bytes, b_bytes, b;      // b: bytes to the tile's first column
  int a_rows, nk;                    // rows of A that count (nobody looks at the others); steps: even, at least 4
};

struct GemmRing {
  static constexpr int kPer = 2;     // requests of a wave per operand and step
  int lane, wave;
  uint32_t lds, b_step, b_two_rows, b_lane[kPer];

  // ldb: row pitch of B
  __device__ __forceinline__ GemmRing(int64_t ldb, const uint16_t* smem) {
    lane = threadIdx.x & 63;
    wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    lds = __builtin_amdgcn_readfirstlane(lds_address(smem));
    b_step = uint32_t(kStepK * ldb * 2);
    b_two_rows = uint32_t(2 * ldb * 2);
    // request j of wave w covers rows 4 w + 2 j and the next: lane l takes 16-byte piece l % 32 of row l / 32, whose 32-byte
    // segments are XORed with f(row)
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      const int row = wave * 4 + 2 * j + (lane >> 5);
      const uint32_t f = uint32_t(row & 3) | uint32_t(row >> 3 & 1) << 2;
      b_lane[j] = uint32_t(int64_t(lane >> 5) * ldb * 2) + (((lane & 31) >> 1) ^ f) * 32 + (lane & 1) * 16;
    }
  }

  // Requests step kt: wave w blocks 2 w and 2 w + 1 of A and rows 4 w .. 4 w + 3 of B.
  __device__ __forceinline__ void issue(const RingSrc& t, rsrc_words_t ra, rsrc_words_t rb, int kt) const {
    const uint32_t to = lds + uint32_t(kt & (kRing - 1)) * kStepBytes + wave * (kPer * 1024);
    // past every operand's end (which lies below 4 GiB by more than that), which gives zeros and moves nothing
    const uint32_t a = wave * 32 < t.a_rows ? uint32_t(kt >> 1) * (kSlabElems * 2) + uint32_t(kt & 1) * 1024 + wave * 4096 : ~0u - 8191;
    const uint32_t b = t.b + uint32_t(kt) * b_step + uint32_t(wave) * (kPer * b_two_rows);
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
      request_lds16(ra, to + j * 1024, lane * 16 + (a + j * 2048));
      request_lds16(rb, to + kTile * kStepK * 2 + j * 1024, b_lane[j] + (b + j * b_two_rows));
    }
  }

  // Until the wave has no more than N requests on their way and its own LDS reads are done, then the others as well.
  template <int N> __device__ __forceinline__ void landed() const {
    static_assert(N < 16, "four bits");
    AERO_CFENCE();
    __builtin_amdgcn_s_waitcnt(0x0070 | N);
    slice_barrier();
  }

  // acc = the tile's product.  active == false: all of the wave's rows (columns) are padding, it only moves operands.
  __device__ __forceinline__ void run(const RingSrc& t, const WavePos& pos, const uint16_t* smem, Acc& acc) const {
    constexpr int kStep = 2 * kPer;   // requests per step
    static_assert(kRing == 4, "the last steps below");
    const int nk = t.nk;
    acc_zero(acc);
    const rsrc_words_t ra = rsrc_words(t.a_base, t.a_bytes), rb = rsrc_words(t.b_base, t.b_bytes);
    descriptors_settled(ra, rb);
#pragma unroll
    for (int kt = 0; kt < kRing - 1; ++kt) issue(t, ra, rb, kt);
    landed<2 * kStep>();
    if (!pos.active) {   // uniform over the wave
      for (int kt = 0; kt < nk - 3; ++kt) {
        issue(t, ra, rb, kt + 3);
        landed<2 * kStep>();
      }
      landed<kStep>();
      landed<0>();
      return;
    }
    const uint32_t fa0 = lds + pos.wm * 8 * 1024 + lane * 16;
    const FragAddr<4> fb0 = frag_addr_bt(smem + kTile * kStepK, pos.wn * 64, lane);
    Frags a1, b_even, b_odd;   // a1, b_odd: of the step before step 0
#pragma unroll
    for (int i = 0; i < kFragBlocks; ++i) a1[i] = b_odd[i] = bf16x8_t{};
    // Step kt, whose operands have landed; the order is pinned.
    auto step = [&](int kt, Frags& b, const Frags& b_before, bool more) {
      constexpr int kMfma = 0x008, kDsRd = 0x100;
      const uint32_t at = uint32_t(kt & (kRing - 1)) * kStepBytes;
      uint32_t fa = fa0 + at;
      asm volatile("" : "+v"(fa));   // one address, the blocks in the instructions' offsets
      FragAddr<4> fb;
      Frags a0;
#pragma unroll
      for (int i = 0; i < kFragBlocks; ++i) {
        a0[i] = lds_fragment(fa + i * 1024);
        fb.at[i] = fb0.at[i] + at;
      }
      frags_load(b, fb, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      frags_mma<true>(a1, b_before, 1, acc);
      __builtin_amdgcn_sched_barrier(0);
      if (more) issue(t, ra, rb, kt + 3);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < kFragBlocks; ++i) a1[i] = lds_fragment(fa + (kFragBlocks + i) * 1024);
      frags_mma<true>(a0, b, 0, acc);
#pragma unroll
      for (int r = 0; r < kFragBlocks; ++r) {
        __builtin_amdgcn_sched_group_barrier(kMfma, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kDsRd, 1, 0);
      }
      __builtin_amdgcn_sched_group_barrier(kMfma, kFragBlocks * (kNB - 1), 0);
      __builtin_amdgcn_sched_barrier(0);   // what follows stays behind the last matrix instruction
    };
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): see GemmStream
    int kt = 0;
#pragma unroll 1
    for (; kt < nk - 4; kt += 2) {
      step(kt, b_even, b_odd, true);
      landed<2 * kStep>();
      step(kt + 1, b_odd, b_even, true);
      landed<2 * kStep>();
    }
    step(kt, b_even, b_odd, true);
    landed<2 * kStep>();
    step(kt + 1, b_odd, b_even, false);
    landed<kStep>();
    step(kt + 2, b_even, b_odd, false);
    landed<0>();
    step(kt + 3, b_odd, b_even, false);
    frags_mma<true>(a1, b_odd, 1, acc);
  }
};

}  // namespace aero
