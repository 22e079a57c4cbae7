// LM head fused into the softmax statistics, the clipped loss and its gradients: logits
// z = hidden @ weight^T exist only as fp32 MFMA accumulator tiles.
//
// Forward   k_compact_valid  rows that have a target are compacted (padding rows take no part in any
//                            contraction; their outputs are written as zeros) and gathered; when a
//                            backward pass follows, the candidates - rows whose rollout has weight and
//                            advantage, i.e. the set AERO's curation leaves - come first; zy = logit of a
//                            row's sampled token (one H-long dot product)
//           k_fused_stats    tile of z^T (vocab rows x token columns): every lane owns one token column
//                            per block, so the running (offset, sum exp, sum exp*z) is a per-lane
//                            register recurrence with no shuffles.  On the candidates' token tiles it
//                            also leaves P = exp(z - zy) in bf16 in K-slabs, tokens x vocabulary and
//                            vocabulary x tokens, both in fragment order, that
//                            the two gradient contractions read (2 x T x V x 2 bytes are held)
//           k_fused_rows     merges the per-tile partials of a token -> logprob, entropy, lse, and in the same
//                            breath the candidates' loss terms and gradient scalars:
//                            dz = g (onehot - exp(z - lse)) = scale * P with scale = -g exp(logprob)
//                            per token, except the sampled token's own entry, which is written here; the
//                            scale travels with the other operand (dweight) or is applied after the
//                            contraction (dhidden), so z is never formed a second time
// Backward  k_fused_dz       only when that does not apply (an entropy term in the rows, or a sampled
//                            token more than 40 nats below another logit, where P would leave its safe
//                            range): recompute the z^T tile and store dz itself in the same layouts
//           k_hidden_and_loss  hidden rows times their scale, transposed; the loss sum
//           k_gemm_dh        dhidden partials = (P or dz) @ weight   (split-K over the vocabulary, fp32)
//           k_scatter_dh     fp32 partials summed in fixed order, times scale -> bf16 dhidden at the original rows
//           k_gemm_dw        dweight = (P or dz)^T @ (scale * hidden)
//           k_gemm_grads     k_gemm_dh and k_gemm_dw in one launch, where either leaves CUs idle
//           k_scatter_and_sum  k_scatter_dh and the sum of dweight's parts, where its range may be split (few tiles, kDwSplitTiles)
// All contractions use the same 256 x 256 MFMA tile, both operands K-contiguous but for the weight in k_gemm_dh,
// whose rows are the contraction index and which a transposing LDS read turns; slices are 64 wide, there 32 (GemmRing).  In all but k_gemm_dh (whose split count
// fills the CUs once or twice), the longer k_gemm_dw (kDwTileRows) and forward tiles of many slices (kForwardTileSlices) a workgroup
// per CU walks the tiles.
#include <algorithm>
#include <mutex>

#include "gemm_tile.h"

namespace aero {

constexpr size_t kWsAlign = 256;
inline size_t up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// ------------------------------------------------------------------------------------------
// workspace
// ------------------------------------------------------------------------------------------
struct FusedPlan {
  int64_t T, T_pad;
  int V, V_ld, H, H_pad, tiles_v;
  size_t off_part, off_fidx, off_nf, off_term, off_flag, off_zy, off_pos, off_nact, off_gc, off_lsec, off_yc, off_ac, off_bc, off_scale,
      off_hc, off_hTc, off_dz, off_dzT, off_dhacc, total;
};

// dhidden is formed as S split-K partials of the active rows, S chosen on the device so that
// (candidate token tiles) x (H tiles) x S fills the launch grid in whole rounds; the buffer holds S
// stacked copies of the active rows, never more rows than the launch grid covers.  A split's weight rows are
// addressed with 32-bit byte offsets.  The rule asks for at most 4 GiB per split of a matrix of T_pad or H_pad columns,
// whichever are more (rows_max), and the grid leaves room for that many splits (plus one) when every token is active.  For the
// addresses H_pad alone would do: with it 32768 tokens take one split instead of three, which measured 0 to 0.9 % of
// a call, and the whole vocabulary would be one chain of fp32 additions.
constexpr int kDhGridMin = 4096;
constexpr int64_t kOperandBytes = int64_t(1) << 32;
static int dh_grid(int64_t T_pad, int H, int V_ld) {
  const int tiles_h = (H + kTile - 1) / kTile;
  const int64_t all = (T_pad / kTile) * tiles_h;
  const int64_t rows = T_pad > int64_t(tiles_h) * kTile ? T_pad : int64_t(tiles_h) * kTile;
  const int64_t s_min = (int64_t(V_ld) * rows * 2 + kOperandBytes - 1) / kOperandBytes;
  const int64_t need = all * (s_min + 1);
  return int(need > kDhGridMin ? need : kDhGridMin);
}
static int64_t dh_part_rows(int64_t T_pad, int H, int V_ld) {
  const int tiles_h = (H + kTile - 1) / kTile;
  const int64_t by_grid = int64_t(dh_grid(T_pad, H, V_ld) / tiles_h + 1) * kTile;   // S x active tiles x H tiles <= grid
  const int64_t by_cap = 64 * T_pad;                                                // S <= 64
  return by_grid < by_cap ? by_grid : by_cap;                                       // >= S * active rows for every S
}

static FusedPlan make_plan(int64_t T, int V, int H) {
  FusedPlan p{};
  p.T = T;
  p.T_pad = int64_t(up(size_t(T > 0 ? T : 1), kTile));
  p.V = V;
  p.V_ld = int(up(size_t(V), kTile));
  p.H = H;
  p.H_pad = int(up(size_t(H), kTile));
  p.tiles_v = p.V_ld / kTile;
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up(bytes, kWsAlign); return at; };
  p.off_part = take(size_t(3) * p.tiles_v * p.T_pad * 4);
  p.off_fidx = take(size_t(p.T_pad) * 4);
  p.off_nf = take(16);
  p.off_term = take(size_t(p.T_pad) * 4);
  p.off_flag = take(size_t(p.T_pad) * 4);
  p.off_zy = take(size_t(p.T_pad) * 4);
  p.off_pos = take(size_t(p.T_pad) * 4);
  p.off_nact = take(20);
  p.off_gc = take(size_t(p.T_pad) * 4);
  p.off_lsec = take(size_t(p.T_pad) * 4);
  p.off_yc = take(size_t(p.T_pad) * 4);
  p.off_ac = take(size_t(p.T_pad) * 4);
  p.off_bc = take(size_t(p.T_pad) * 4);
  p.off_scale = take(size_t(p.T_pad) * 4);
  p.off_hc = take(size_t(p.T_pad) * H * 2);
  p.off_hTc = take(size_t(p.H_pad) * p.T_pad * 2);
  p.off_dz = take(size_t(p.T_pad) * p.V_ld * 2);
  p.off_dzT = take(size_t(p.V_ld) * p.T_pad * 2);
  p.off_dhacc = take(size_t(dh_part_rows(p.T_pad, H, p.V_ld)) * H * 4);
  p.total = o;
  return p;
}

size_t fused_workspace_bytes(int64_t T, int32_t V, int32_t H) {
  if (T < 0 || V < 1 || H < 1) return 0;
  return make_plan(T, V, H).total;
}

// Split-K factor for dhidden, from the number of candidate token tiles (device side; one wave, lane s - 1
// prices s splits).  A workgroup's time is its share of the K slices plus a fixed tail (storing its fp32
// partial tile, worth about 8 slices of main loop); the launch takes ceil(workgroups / 256) such rounds.
// S minimises rounds x (slices / S + 8) among the S whose splits are small enough (see dh_grid): a split's
// range times rows_max columns of bf16 must stay below 4 GiB.  Chosen once per call: the
// 64-bit divisions are 50 us of latency when one thread walks the candidates, and every workgroup of
// the contraction and of the scatter used to (400 of the 530 us of the contraction of 600 tokens).
__device__ __forceinline__ int dh_splits(int active_tiles, int tiles_h, int grid, int slices, int64_t rows_max) {
  const int base = active_tiles * tiles_h;
  if (base == 0) return 0;
  const int s = int(threadIdx.x & 63) + 1;
  const int per = (slices + s - 1) / s;
  const bool ok = int64_t(base) * s <= grid && s <= slices && int64_t(per) * kDK * rows_max * 2 < (int64_t(1) << 32);
  const int64_t cost = (int64_t(base) * s + 255) / 256 * (per + 8);
  int64_t best = ok ? cost * 64 + (s - 1) : INT64_MAX;   // the fewest splits among equals
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) best = min(best, int64_t(__shfl_xor((long long)best, off, kWave)));
  return best == INT64_MAX ? 0 : int(best & 63) + 1;
}

// A gradient dweight of few tiles leaves CUs idle however many tokens there are: up to kDwSplitTiles tiles the candidates' range
// is split into parts, whose sums lie in fp32 behind the dhidden partials until k_scatter_and_sum adds them up in order.
// Whether it pays depends on the candidates, which only the device knows, and on the tiles: one range takes as long as its slices
// unless dhidden's workgroups fill the idle CUs meanwhile (k_gemm_grads), and with half the CUs' number of tiles they do; the parts' way to
// memory and back has to be shorter than what is left.  So the host says what may be (most, from the rows) and dw_parts decides,
// by a line through the counts at which the two came out even.  Whole calls, one range / split, by tiles: 16 (H = 64, V = 4000) 1125 candidates 73.1 / 63.4 us, 4750 162 / 99; 32 (256, 8000) 1125 97.7 / 87.0; 48
// (512, 6144) 1125 102.5 / 94.9; 57 (640, 4753) 1437 101.5 / 105.4, 2125 137 / 132; 64 (1024, 4096) 1437 113.6 / 113.5, 2125 145.4 / 138.4; 72
// (424, 9000) 2125 140.0 / 138.9, 4750 248.5 / 237.7; 85 (256, 21760) 3000 235 / 241, 4750 326 / 323, 7500 482 / 463; 96 (768, 8192) 4750
// 274 / 280, 7500 408 / 397; 112 (1792, 4096) 4750 284 / 301, 12500 709 / 709; 128 (896, 8000) 4750 292 / 296, 12500 727 / 720.  (Decided by the
// rows alone, calls of 1300 to 2700 rows with 40 to 65 % of them candidates had one part, and lost 2 to 7 % by its detour.)
constexpr int kDwSplitTiles = 128, kDwSplitMax = 16;
constexpr int kDwSplitSlices = 8;   // of a part, at least, but for the last
struct DwSplit {
  int most, tiles, V;   // parts at most; tiles of the gradient
  int64_t rows;         // of the dhidden partials' buffer
};
__host__ __device__ inline bool dw_split_pays(int tiles, int64_t slices) {
  return slices >= 2 * kDwSplitSlices && 2 * slices >= 3 * (tiles - 42);
}
__device__ __forceinline__ int dw_parts(const DwSplit& q, int n_cand, int dh_splits) {
  const int slices = (n_cand + kDK - 1) / kDK, parts = min(q.most, slices / kDwSplitSlices);
  const int64_t left = q.rows - int64_t(dh_splits) * ((n_cand + kTile - 1) / kTile * kTile);
  if (parts < 2 || !dw_split_pays(q.tiles, slices) || left < int64_t(parts) * q.V) return 1;
  const int per = (slices + parts - 1) / parts;
  return (slices + per - 1) / per;   // none of them empty (97 slices in 12 parts are ten of 9, one of 7 and nothing)
}

// Where the parts lie: behind the dhidden partials.
__device__ __forceinline__ int64_t dw_part_offset(const int32_t* nact, int H) { return int64_t(nact[3]) * nact[1] * H; }

// ------------------------------------------------------------------------------------------
// forward: rows with a target, compacted
// ------------------------------------------------------------------------------------------
// Rows without a target (padding) take no part in the contraction.  Single workgroup, order-preserving
// inside each of two classes: first the candidates - rows that may carry gradient, which is known before the
// forward pass: a target in [0, V), a rollout index in [0, R), weight != 0 and (advantage != 0 or
// every_weighted: an entropy or KL term is on) - then the other rows with a target.
//   fidx[j] = row of position j (-1 past the count), nf = {rows with a target, that rounded up to a tile,
//   candidates, that rounded up to a tile}; pos[t] = position of candidate t, -1 for every other row;
//   nact = {candidates, rounded up, 0, splits, parts}: nact[2] is the flag the forward pass raises when a stored
//   exponential left its safe range (see k_fused_stats), nact[3] the split count of the dhidden contraction, nact[4]
//   the part count of dweight's.
// token_rollout == null (forward-only call): no candidates, pos / nact are not written.
// Ignored rows get their zero outputs here; a target >= V or a rollout index >= R raises its device error bit.
template <int kAhead>
__global__ __launch_bounds__(1024) void k_compact_valid(
    const int32_t* __restrict__ targets, int64_t T, int64_t T_pad, int V, const int32_t* __restrict__ token_rollout,
    const float* __restrict__ adv, const float* __restrict__ weight, int R, int every_weighted,
    int32_t* __restrict__ fidx, int32_t* __restrict__ nf, int32_t* __restrict__ pos, int32_t* __restrict__ nact,
    float* __restrict__ logprob, float* __restrict__ entropy, float* __restrict__ lse_out,
    int32_t* __restrict__ err_flag, int tiles_h, int dh_grid, int slices, int64_t rows_max, DwSplit split) {
  // Each of the 16 waves owns one contiguous range of rows, 64 at a time (coalesced reads, ballot + popcount inside the
  // wave): count, exchange the 16 counts, then place.  Latency bound: the loads of kAhead steps go out together, those that need
  // another's answer from clamped positions so that no branch stands between them, and the first kKept steps' classes stay in
  // a register for the second time.  (Steps one by one, their loads one behind the other and all of it twice / this way: 600 rows 4.2 / 3.5 us,
  // 2048 6.2 / 5.3, 4096 9.9 / 5.8, 8192 17.0 / 8.4, 16384 31.8 / 14.0, 32768 64.3 / 25.3, 40000 96.2 / 34.9; eight or sixteen steps at a
  // time 13.7 and 14.4 for 16384: the code, which comes from memory once per launch, grows with them.)
  constexpr int kKept = 32;
  static_assert(kKept % kAhead == 0, "whole blocks of steps");
  __shared__ int wsum_c[16], wsum_o[16];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int64_t seg = ((T + 15) / 16 + 63) / 64 * 64;
  const int64_t lo = min(T, wave * seg), hi = min(T, lo + seg);
  const uint64_t below = (uint64_t(1) << lane) - 1;
  bool bad_y = false, bad_i = false;
  // classes of the rows lo + 64 (it + u) + lane: 0 = no target, 1 = target only, 2 = candidate
  auto classes = [&](int it, int (&cls)[kAhead]) {
    int y[kAhead], i[kAhead];
    float w[kAhead], A[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int64_t t = min(lo + int64_t(it + u) * 64 + lane, T - 1);
      y[u] = targets[t];
      i[u] = token_rollout ? token_rollout[t] : -1;
    }
    const bool rollouts = token_rollout && R > 0;   // uniform
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int at = min(max(i[u], 0), R - 1);
      w[u] = rollouts ? weight[at] : 0.f;
      A[u] = rollouts ? adv[at] : 0.f;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const bool in = lo + int64_t(it + u) * 64 + lane < hi, target = in && unsigned(y[u]) < unsigned(V);
      const bool rollout = i[u] >= 0 && i[u] < R;
      cls[u] = !target ? 0 : rollout && w[u] != 0.f && (every_weighted || A[u] != 0.f) ? 2 : 1;
      bad_y |= in && y[u] >= V;
      bad_i |= in && y[u] >= 0 && i[u] >= R;
    }
  };
  const int steps = int((hi - lo + 63) / 64);
  uint64_t kept = 0;
  int cnt_c = 0, cnt_o = 0;
  for (int it = 0; it < steps; it += kAhead) {
    int cls[kAhead];
    classes(it, cls);
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      cnt_c += __popcll(__ballot(cls[u] == 2));
      cnt_o += __popcll(__ballot(cls[u] == 1));
      if (it < kKept) kept |= uint64_t(cls[u]) << (2 * (it + u));
    }
  }
  if (lane == 0) {
    wsum_c[wave] = cnt_c;
    wsum_o[wave] = cnt_o;
  }
  __syncthreads();
  int run_c = 0, run_o = 0, total_c = 0, total_o = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    run_c += w < wave ? wsum_c[w] : 0;
    run_o += w < wave ? wsum_o[w] : 0;
    total_c += wsum_c[w];
    total_o += wsum_o[w];
  }
  run_o += total_c;   // the other rows follow the candidates
  const int total = total_c + total_o;
  for (int it = 0; it < steps; it += kAhead) {
    int cls[kAhead];
    if (it < kKept) {   // uniform
#pragma unroll
      for (int u = 0; u < kAhead; ++u) cls[u] = int(kept >> (2 * (it + u))) & 3;
    } else {
      classes(it, cls);
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int64_t t = lo + int64_t(it + u) * 64 + lane;
      const bool in = t < hi;
      const uint64_t m_c = __ballot(cls[u] == 2), m_o = __ballot(cls[u] == 1);
      int at = -1;
      if (cls[u] == 2) {
        at = run_c + __popcll(m_c & below);
        fidx[at] = int(t);
      } else if (cls[u] == 1) {
        fidx[run_o + __popcll(m_o & below)] = int(t);
      } else if (in) {
        logprob[t] = 0.f;
        lse_out[t] = 0.f;
        if (entropy) entropy[t] = 0.f;
      }
      if (in && pos) pos[t] = at;
      run_c += __popcll(m_c);
      run_o += __popcll(m_o);
    }
  }
  if ((bad_y || bad_i) && err_flag)
    atomicOr(err_flag, (bad_y ? AERO_DERR_BAD_TARGET : 0) | (bad_i ? AERO_DERR_BAD_ROLLOUT : 0));
  for (int64_t j = total + tid; j < T_pad; j += 1024) fidx[j] = -1;
  const int splits = wave == 0 && nact ? dh_splits((total_c + kTile - 1) / kTile, tiles_h, dh_grid, slices, rows_max) : 0;
  if (tid == 0) {
    nf[0] = total;
    nf[1] = (total + kTile - 1) / kTile * kTile;
    nf[2] = total_c;
    nf[3] = (total_c + kTile - 1) / kTile * kTile;
    if (nact) {
      nact[0] = total_c;
      nact[1] = (total_c + kTile - 1) / kTile * kTile;
      nact[2] = 0;
      nact[3] = splits;
      nact[4] = dw_parts(split, total_c, splits);
    }
  }
}

// Row j of `out` = hidden row fidx[j] (zeros where fidx[j] < 0), and zy[j] = logit of its sampled token = <hidden
// row, weight row>, fp32 accumulation of the bf16 products in a fixed order (0 past the count).  H % 8 == 0,
// 16-byte vectors; one wave per row, n_rows a multiple of 4.
__global__ __launch_bounds__(256) void k_gather_rows(const uint16_t* __restrict__ in, const uint16_t* __restrict__ W, int H,
                                                     const int32_t* __restrict__ fidx,
                                                     const int32_t* __restrict__ targets, uint16_t* __restrict__ out,
                                                     float* __restrict__ zy) {
  const int lane = threadIdx.x & 63;
  const int64_t j = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
  const int src = fidx[j];
  const uint16_t* hr = in + int64_t(max(src, 0)) * H;
  const uint16_t* wr = W + int64_t(src >= 0 ? targets[src] : 0) * H;   // 0 <= target < V by construction of fidx
  float dot = 0.f;
  for (int k = lane * 8; k < H; k += kWave * 8) {
    u32x4_t v = {0u, 0u, 0u, 0u};
    if (src >= 0) {
      v = *reinterpret_cast<const u32x4_t*>(hr + k);
      float a[8], b[8];
      unpack8(v, a);
      unpack8(*reinterpret_cast<const u32x4_t*>(wr + k), b);
#pragma unroll
      for (int e = 0; e < 8; ++e) dot = fmaf(a[e], b[e], dot);
    }
    *reinterpret_cast<u32x4_t*>(out + j * H + k) = v;
  }
  dot = wave_reduce(dot, [](float x, float y) { return x + y; });
  if (lane == 0) zy[j] = dot;
}

// A 256 x 256 bf16 tile (vocabulary rows m0.., token columns n0..) held as packed pairs in the accumulator
// layout, pk[nb][mb] = the four rows acc_row(wm, mb, 0 .. 3) of column acc_col(wn, nb), leaves in the two
// layouts the gradient contractions read, both K-slabs in fragment order (frag_order_offset): tokens x vocabulary, and
// vocabulary x tokens.  Every instruction stores one 1 KB block, so nothing is staged in LDS and no wave
// waits for another.  A block is turned round by the matrix unit: its registers are also the left operand
// of a 16 x 16 x 16 instruction (rows = tokens), and times the identity it comes back exactly with the tokens in a lane's
// registers and the vocabulary across the lanes - one instruction and two conversions in place of some twenty exchanges and
// selections between lanes.
constexpr int kTileStores = 2 * kNB * kMB / 2;   // per wave
__device__ __forceinline__ void store_tile_both_layouts(const uint32_t (&pk)[kNB][kMB][2], const WavePos& wp, int lane, int m0, int n0,
                                                        int64_t T_pad, int V_ld, uint16_t* __restrict__ dz, uint16_t* __restrict__ dzT) {
  typedef short s16x4_t __attribute__((ext_vector_type(4)));
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  const int group = lane >> 4;
  constexpr int kNonTemporal = 2;
  // Two neighbouring blocks along K: the odd 16-lane rows of the first change places with the even ones of the second; lane
  // group 0 then holds K 0..7 of its row, group 2 8..15, group 1 16..23, group 3 24..31.
  auto store = [&](__amdgpu_buffer_rsrc_t to, const u32x2_t& first, const u32x2_t& second, uint32_t lane_off, uint32_t off) {
    const auto lo = __builtin_amdgcn_permlane16_swap(first.x, second.x, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap(first.y, second.y, false, false);
    // The whole offset in the vector register: with a part of it in a scalar one the compiler writes the data registers
    // again in the very next instruction, and some lanes stored the values of the block behind.
    __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{lo[0], hi[0], lo[1], hi[1]}, to, lane_off + off, 0, kNonTemporal);
  };
  const uint32_t in_block = uint32_t((lane & 15) * 8 + ((group & 1) * 2 + (group >> 1)) * 128) * 2;   // row lane % 16, that K
  // ---- tokens x vocabulary: four slabs of a token tile, the wave's 128 vocabulary rows are two of them ----
  constexpr uint32_t slab = kSlabElems * 2;   // bytes
  const __amdgpu_buffer_rsrc_t rz =
      __builtin_amdgcn_make_buffer_rsrc(dz + slab_offset(V_ld / 64, n0 / kTile, m0 / 64), 0, int(4 * slab), 0x00020000);
  const uint32_t at = uint32_t(wp.wn * 64) * 128 + wp.wm * 2 * slab;
#pragma unroll
  for (int nb = 0; nb < kNB; ++nb)
#pragma unroll
    for (int mb = 0; mb < kMB; mb += 2)
      store(rz, u32x2_t{pk[nb][mb][0], pk[nb][mb][1]}, u32x2_t{pk[nb][mb + 1][0], pk[nb][mb + 1][1]}, in_block,
            at + (mb / 4) * slab + (mb / 2 % 2) * 1024 + nb * 2048);
  // ---- vocabulary x tokens: four slabs of a vocabulary tile, the wave's 64 tokens are one of them ----
  const __amdgpu_buffer_rsrc_t rzT =
      __builtin_amdgcn_make_buffer_rsrc(dzT + slab_offset(T_pad / 64, m0 / kTile, n0 / 64), 0, int(4 * slab), 0x00020000);
  const uint32_t atT = uint32_t(wp.wm * 128) * 128 + wp.wn * slab;
  const int diag = (lane & 15) - 4 * group;   // the lane's register of the identity that is 1
  const u32x2_t one = {diag == 0 ? 0x3f80u : diag == 1 ? 0x3f800000u : 0u, diag == 2 ? 0x3f80u : diag == 3 ? 0x3f800000u : 0u};
  auto turned = [&](const uint32_t (&block)[2]) {
    const f32x4_t t = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, u32x2_t{block[0], block[1]}),
                                                                __builtin_bit_cast(s16x4_t, one), f32x4_t{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    return u32x2_t{pack_bf16x2(t.x, t.y), pack_bf16x2(t.z, t.w)};
  };
#pragma unroll
  for (int mb = 0; mb < kMB; ++mb)
#pragma unroll
    for (int nb = 0; nb < kNB; nb += 2)
      store(rzT, turned(pk[nb][mb]), turned(pk[nb + 1][mb]), in_block, atT + mb * 2048 + (nb / 2) * 1024);
}

// ------------------------------------------------------------------------------------------
// forward: per-tile softmax partials
// ------------------------------------------------------------------------------------------
// grid: xcd_grid(tiles_v * T_pad / 256) workgroups, at most one per CU unless tiles are long (kForwardTileSlices).  Hf holds the compacted rows ([T_pad][H], zero
// past the count); part_* are [tiles_v][T_pad], indexed by compact row.
//
// STORE (a backward pass follows and its rows have the plain form dz = g (onehot - pi)): the token tiles that
// hold candidates also leave P = exp(z - zy) in bf16, zy = the sampled token's own logit (k_gather_rows), in
// the two K-slab layouts of the gradient contractions, so that the backward pass need not form z again:
//   dz[t, v] = s_t P[t, v] (v != y_t),  s_t = -g_t exp(logprob_t),  because exp(z - lse) = exp(z - zy) exp(zy - lse);
// the per-token factor s_t moves into the other operand (dweight) or behind the contraction (dhidden), and the
// one entry per row that differs, v = y_t, is overwritten once the log-prob is known (candidate_row).
// bf16 keeps fp32's exponent range, so P is safe as long as z - zy stays far below 88, and so is the scale
// (about g times the sampled token's probability, which must stay a normal number after it is multiplied
// into a bf16 hidden row) as long as that probability is not below e^-52 or so; a tile that sees
// z - zy > kStoreRange on a candidate column raises nact[2], and the backward pass then forms dz by
// recomputing z as it does for rows with an entropy term (k_fused_dz).  The exponentials are the ones the
// statistics take anyway: P = exp(z - m) * exp(m - zy) with m the running offset of the lane.
// What a ragged token tile does not hold costs little: rows past the count lie behind the operand's bytes (a request for them
// moves nothing), a wave without a row has no epilogue, 64 columns without a candidate are not stored, and the dhidden
// contraction does not request 32 rows without one.  Whole calls at H = 1536, V = 151936: 100 tokens 462 -> 428 us, 300 602 -> 572,
// 600 776 -> 761; forward only 300 tokens 235 -> 215; 1100 tokens at H = 896, V = 50257 348 -> 333.
constexpr float kStoreRange = 40.f;

// From so many K slices on the forward contraction and the recomputation have a workgroup per tile, as the long dweight has.
// Forward-only calls, walking / per tile: H = 3584 4000 tokens 3274 / 3306 us, 600 711 / 704, 16384 (V = 152064) 13.50 / 13.26 ms; H = 4096 700
// tokens 675 / 681, 4096 3170 / 3200, 16384 6294 / 6327; H = 4352 300 tokens 436 / 439, 600 894 / 808, 1400 1299 / 1244, 8000 6595 / 6432; H = 5120
// 600 tokens 1106 / 958, 1400 1731 / 1707, 8000 9615 / 9108; H = 7168 1000 tokens 1748 / 1495; H = 8192 300 tokens 745 / 748, 3000 4715 / 4729,
// 16000 6618 / 6255.
constexpr int kForwardTileSlices = 65;

// stat_update for 16 values that also hands back the exponentials it formed (relative to st.m on return)
// and the largest of the 16 values.
__device__ __forceinline__ float stat_update_keep(RowStat& st, const float (&z)[16], float (&e)[16]) {
  float vm = z[0];
#pragma unroll
  for (int k = 1; k + 1 < 16; k += 2) vm = max3(vm, z[k], z[k + 1]);
  vm = fmaxf(vm, z[15]);
  const bool grow = vm > st.m + kLazy;
  if (__builtin_amdgcn_ballot_w64(grow) != 0) {
    asm volatile("" ::: "memory");
    if (grow) {
      const float f = (st.m == -INFINITY) ? 0.f : exp2_fast((st.m - vm) * kLog2e);
      st.s *= f;
      st.sz *= f;
      st.m = vm;
    }
  }
  const float c = -st.m * kLog2e;
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    e[k] = exp2_fast(fmaf(z[k], kLog2e, c));
    st.s += e[k];
    st.sz = fmaf(e[k], z[k], st.sz);
  }
  return vm;
}

template <bool STORE>
__global__ __launch_bounds__(kGemmNT, 2) void k_fused_stats(
    const uint16_t* __restrict__ W, const uint16_t* __restrict__ Hf, int V, int H, int tiles_v,
    int64_t T_pad, const int32_t* __restrict__ nf, float* __restrict__ part_m,
    float* __restrict__ part_s, float* __restrict__ part_sz, const float* __restrict__ zy, int V_ld,
    int32_t* __restrict__ nact, uint16_t* __restrict__ dz, uint16_t* __restrict__ dzT) {
  extern __shared__ __align__(16) uint16_t smem[];
  // the tile order covers only the token tiles that hold rows with a target (count known on the
  // device), so that every XCD gets the same number of real tiles
  const int tiles_t_act = nf[1] / kTile, n_rows = nf[0], n_cand = STORE ? nf[2] : 0;
  const int n_tiles = tiles_v * tiles_t_act;
  const int lane = threadIdx.x & 63;
  WavePos wp = wave_pos<true>();
  const int wm = wp.wm, wn = wp.wn;
  GemmStream<true, false, false, true> stream(H, kDK, H, kDK, H);
  auto source = [&](int tv, int tt) {
    return TileSrc{W, Hf, (int64_t(V) * H) * 2, (int64_t(n_rows) * H) * 2, uint32_t(int64_t(tv) * kTile * H * 2),
                   uint32_t(int64_t(tt) * kTile * H * 2), (H + kDK - 1) / kDK};
  };
  RowStat* const xch = reinterpret_cast<RowStat*>(smem + kEpilogueOff / 2);   // [256 token columns]
  // zy of a tile's columns, sent to LDS right behind its first slice: a load in the epilogue would wait for everything
  // that the next tile has requested by then.  Two buffers, taken in turn.
  float* const ref_buf = reinterpret_cast<float*>(xch + kTile);
  auto request_ref = [&](int tt, int buf) {
    if (!STORE || stream.wave >= kTile / kWave) return;
    const __amdgpu_buffer_rsrc_t rz = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(zy), 0, int(T_pad * 4), 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rz, ref_buf + buf * kTile + stream.wave * kWave, 4,
                                             uint32_t(tt * kTile + stream.wave * kWave + lane) * 4, 0, 0, 0);
  };
  int pid = blockIdx.x, tv, tt, buf = 0;
  bool more = tile_of_step(pid, tiles_v, tiles_t_act, 0, n_tiles, tv, tt), stored = false;
  if (!more) return;   // uniform over the workgroup
  TileSrc src = source(tv, tt);
  stream.start(src, smem);
  request_ref(tt, buf);
  while (more) {
    const int m0 = tv * kTile, n0 = tt * kTile;
    const bool store = STORE && n0 + wn * 64 < n_cand;   // uniform over the wave: nobody reads 64 columns without a candidate
    wp.active = n0 + wn * 64 < n_rows;
    const bool active = !STORE || wp.active;   // the epilogue has something to do (without the stores the branch costs what it saves)
    wp.warm_a = warm_share(tt, tiles_t_act);
    wp.warm_b = warm_share(tv, tiles_v);
    wp.warm_from = forward_warm_from(tiles_t_act);
    const int tv_now = tv;
    pid += gridDim.x;
    more = tile_of_step(pid, tiles_v, tiles_t_act, 0, n_tiles, tv, tt);
    const TileSrc next = more ? source(tv, tt) : no_tile(src);
    Acc acc;
    stream.run<kTileStores>(src, next, wp, stored, smem, acc);
    src = next;
    stored = store;
    request_ref(tt, buf ^ 1);

    const int lane = opaque(threadIdx.x & 63);
    const bool full = m0 + kTile <= V;
    uint32_t pk[kNB][kMB][2] = {};   // a value on every path: not carried around the walk
    bool wide = false;
    const int my_col = acc_col(wn, (lane & 16 ? 2 : 0) + (lane & 32 ? 1 : 0), lane);
    RowStat mine = stat_identity();
    if (active) {   // uniform over the wave
      RowStat st[kNB];
      constexpr int kGroup = 4;   // accumulator blocks per statistics update: 16 values
#pragma unroll
      for (int nb = 0; nb < kNB; ++nb) {
        st[nb] = stat_identity();
        const int col = n0 + acc_col(wn, nb, lane);
        const bool col_cand = store && col < n_cand;
        const float ref = store ? ref_buf[buf * kTile + acc_col(wn, nb, lane)] : 0.f;
#pragma unroll
        for (int mg = 0; mg < kMB; mg += kGroup) {
          if (full) {
            float z[16], e[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) z[i] = acc[mg + i / 4][nb][i % 4];
            if (store) {
              const float vm = stat_update_keep(st[nb], z, e);
              // columns past the candidates keep zeros: their rows of the other operand are zero as well
              const float f = col_cand ? exp2_fast((st[nb].m - ref) * kLog2e) : 0.f;
              wide |= col_cand && vm - ref > kStoreRange;
#pragma unroll
              for (int k = 0; k < kGroup; ++k) {
                pk[nb][mg + k][0] = pack_bf16x2(e[4 * k] * f, e[4 * k + 1] * f);
                pk[nb][mg + k][1] = pack_bf16x2(e[4 * k + 2] * f, e[4 * k + 3] * f);
              }
            } else {
              stat_update<16>(st[nb], z);
            }
          } else {
            float d[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              d[i] = 0.f;
              if (m0 + acc_row(wm, mg + i / 4, i % 4, lane) < V) {
                const float zi = acc[mg + i / 4][nb][i % 4];
                float z[1] = {zi};
                stat_update<1>(st[nb], z);
                if (store && col_cand) {
                  d[i] = exp2_fast((zi - ref) * kLog2e);
                  wide |= zi - ref > kStoreRange;
                }
              }
            }
            if (store) {
#pragma unroll
              for (int k = 0; k < kGroup; ++k) {
                pk[nb][mg + k][0] = pack_bf16x2(d[4 * k], d[4 * k + 1]);
                pk[nb][mg + k][1] = pack_bf16x2(d[4 * k + 2], d[4 * k + 3]);
              }
            }
          }
        }
      }
      // Four lanes (l % 16 equal) share a column and hold the same four columns each: two exchanges in which a
      // lane passes on half of its columns leave every lane with one of the wave's 64 columns, whole.
      static_assert(kNB == 4, "the exchange below halves four columns twice");
      const bool hi16 = lane & 16, hi32 = lane & 32;
      RowStat two[2];
#pragma unroll
      for (int k = 0; k < 2; ++k)
        two[k] = stat_merge(hi16 ? st[2 + k] : st[k], stat_shfl_xor(hi16 ? st[k] : st[2 + k], 16));
      mine = stat_merge(hi32 ? two[1] : two[0], stat_shfl_xor(hi32 ? two[0] : two[1], 32));
    }
    // the two waves that share these token columns (wm = 0, 1) merge through LDS
    buf ^= 1;
    if (wm == 1 && active) xch[my_col] = mine;
    lds_barrier();   // the slices of the next tile put barriers between these reads and the next writes
    if (wm == 0 && active) {
      const RowStat r = stat_merge(mine, xch[my_col]);
      const int64_t o = int64_t(tv_now) * T_pad + n0 + my_col;   // column < T_pad
      part_m[o] = r.m;
      part_s[o] = r.s;
      part_sz[o] = r.sz;
    }
    if constexpr (STORE) {
      if (store) {
        if (__any(wide) && lane == 0) atomicOr(nact + 2, 1);
        store_tile_both_layouts(pk, wp, lane, m0, n0, T_pad, V_ld, dz, dzT);
      }
    }
  }
  end_of_walk();
}

// ------------------------------------------------------------------------------------------
// per token: statistics, loss term, scalars of the gradient row
// ------------------------------------------------------------------------------------------
// What the backward part needs of a row, all nullptr / unused in a forward-only call.  Per-candidate outputs are in
// candidate order (position j <-> token fidx[j]; positions from the count up to T_pad are padding without
// gradient).  The gradient row of a candidate is
//   dz_v = pi_v (ac z_v + bc) + gc 1[v = y],   (ac, bc) = (0, -g) without an entropy term.
// Two ways to get there, chosen here for the whole call (recompute = the caller forces it, or the forward
// pass raised nact[2]):
//   stored       the forward pass left P = exp(z - zy): dz_v = scale P_v with scale = -g exp(logprob), and the
//                entry v = y, g (1 - pi_y) = scale * (-(exp(-logprob) - 1)), is written into both layouts here
//   recompute    k_fused_dz forms dz from gc / lsec / yc / ac / bc; scale = 1
// scale is 0 on padding positions, so that rows the forward tile stored past the candidates drop out.
struct FusedTerms {
  const int32_t *targets, *token_rollout;
  const float *old_logprob, *adv, *weight, *ref_logprob;
  LossHyper hyper;
  const int32_t* nact;
  int64_t T_pad;
  int V_ld, force_recompute;
  float* term;
  int32_t* flag;
  float *gc, *lsec;
  int32_t* yc;
  float *ac, *bc, *scale;
  uint16_t *dz, *dzT;
};

__device__ __forceinline__ void candidate_row(const FusedTerms& q, int64_t j, int64_t t, float lse, float lp, float low,
                                              float entropy) {
  const int i = q.token_rollout[t], y = q.targets[t];
  const LossHyper& h = q.hyper;
  const float A = q.adv[i], w = q.weight[i];
  TokenTerm r = token_term(h, A, w, lp, low, A != 0.f ? q.old_logprob[t] : 0.f, h.kl_coef != 0.f ? q.ref_logprob[t] : 0.f);
  float ac = 0.f, bc = -r.g;
  if (h.ent_coef != 0.f) {
    r.term -= h.ent_coef * w * entropy;
    ac = h.grad_scale * h.ent_coef * w;
    bc = ac * (entropy - lse) - r.g;
  }
  q.term[j] = r.term;
  q.flag[j] = r.flag;
  q.gc[j] = r.g;
  q.lsec[j] = lse;
  q.yc[j] = y;
  q.ac[j] = ac;
  q.bc[j] = bc;
  if (q.force_recompute || q.nact[2] != 0) {
    q.scale[j] = 1.f;
    return;
  }
  q.scale[j] = -r.g * expf(lp);
  const uint16_t own = f32_to_bf16(-expm1f(-lp));
  q.dz[frag_order_offset(q.V_ld / 64, j, y)] = own;
  q.dzT[frag_order_offset(q.T_pad / 64, y, j)] = own;
}

// TOK consecutive compact rows per workgroup of 1024 threads.  The tiles_v partials of a row are split over
// 1024 / TOK threads, which keep kRowsAhead of them in flight, merged through LDS and a lane reduction.  The
// log-partition and the log-prob are formed in 64 bits: what their rounding to 32 bits leaves off the log-prob
// goes into the ratio, whose terms cancel inside a group.  Results go to the row's original position, and a candidate
// row's loss term and gradient scalars are formed on the spot.  TOK: 64 reads whole 256-byte segments; a few
// hundred tokens are a handful of workgroups that way (16 us at 600 tokens whatever the prefetch), so up to
// kFewRows rows are taken 16 at a time.
constexpr int kRowsNT = 1024, kRowsAhead = 8;
constexpr int64_t kFewRows = 4096;
template <int TOK>
__global__ __launch_bounds__(kRowsNT) void k_fused_rows(
    int tiles_v, int64_t T_pad, const int32_t* __restrict__ fidx, const int32_t* __restrict__ nf,
    const float* __restrict__ part_m, const float* __restrict__ part_s, const float* __restrict__ part_sz,
    const float* __restrict__ zy, float* __restrict__ logprob, float* __restrict__ entropy,
    float* __restrict__ lse_out, FusedTerms q) {
  constexpr int kStreams = kRowsNT / TOK;   // threads per row: 16 or 64
  __shared__ RowStat xs[kStreams][TOK];
  const int tid = threadIdx.x, stream = tid / TOK;
  const int64_t j0 = int64_t(blockIdx.x) * TOK;   // j0 + TOK <= T_pad
  const int n = nf[0];
  const int n_cand = q.nact ? q.nact[0] : 0;
  const int64_t mine = j0 + tid / kStreams;   // the row this thread finishes
  const bool leader = tid % kStreams == 0;
  if (q.nact && leader && mine >= n_cand) {   // padding position of the gradient operands
    q.gc[mine] = 0.f;
    q.lsec[mine] = 1e30f;   // exp(z - lsec) = 0 whatever z is
    q.yc[mine] = -1;
    q.ac[mine] = 0.f;
    q.bc[mine] = 0.f;
    q.scale[mine] = 0.f;
  }
  if (j0 >= n) return;   // uniform over the workgroup
  RowStat st = stat_identity();
  for (int tv = stream; tv < tiles_v; tv += kRowsAhead * kStreams) {
    RowStat v[kRowsAhead];
#pragma unroll
    for (int u = 0; u < kRowsAhead; ++u) {
      const int at = tv + u * kStreams;
      const int64_t o = int64_t(at) * T_pad + j0 + tid % TOK;
      v[u] = at < tiles_v ? RowStat{part_m[o], part_s[o], part_sz[o]} : stat_identity();
    }
#pragma unroll
    for (int u = 0; u < kRowsAhead; ++u) st = stat_merge(st, v[u]);
  }
  xs[stream][tid % TOK] = st;
  __syncthreads();
  const RowStat r = stat_reduce<kStreams == kWave>(xs[tid % kStreams][tid / kStreams]);
  if (!leader || mine >= n) return;
  const int64_t t = fidx[mine];
  const double lse = double(r.m) + log(double(r.s));
  const double lp = double(zy[mine]) - lse;
  const float lp32 = float(lp), lse32 = float(lse), ent = float(lse - double(r.sz) / double(r.s));
  logprob[t] = lp32;
  lse_out[t] = lse32;
  if (entropy) entropy[t] = ent;
  if (mine < n_cand) candidate_row(q, mine, t, lse32, lp32, remainder_of(lp32, float(lp - double(lp32))), ent);
}

// ------------------------------------------------------------------------------------------
// backward: the other operand of dweight, and the loss
// ------------------------------------------------------------------------------------------
// The candidates' hidden rows ([T_pad][H], H % 8 == 0, 16-byte aligned), each times its scale (product in fp32, rounded to
// bf16 once), transposed into the K-slab layout the GEMM tile reads: row r becomes K index r, column c operand row c:
//   out[slab_offset(T_pad / 64, c / 256, r / 64) + c % 256 * 64 + r % 64] = scale[r] * in[r][c]
// for c < C_pad; columns from H on do not exist in `in` and give 0.
// 64 x 64 tiles through LDS, one per workgroup of the grid (T_pad / 64 + 1, C_pad / 64); the first workgroup of the last
// column forms the loss from the candidates' terms meanwhile (a launch of its own: 4.7 us a call).  Every global access is a 16-byte
// vector: the tile is held in LDS as [r][c] with 32-bit writes; a thread then collects 8 consecutive r of one
// column c for one 16-byte store, threads ordered so that a workgroup writes its 64 x 64 block of the slab as one
// contiguous 8 KB run.
__global__ __launch_bounds__(256) void k_hidden_and_loss(const uint16_t* __restrict__ in, int64_t T_pad, int C, int C_pad,
                                                         uint16_t* __restrict__ out, const float* __restrict__ scale,
                                                         const float* __restrict__ term, const int32_t* __restrict__ flag,
                                                         const int32_t* __restrict__ nact, float* __restrict__ loss,
                                                         float* __restrict__ clip_frac) {
  __shared__ uint32_t tile[64][33];   // [r][c / 2]
  const int64_t r0 = int64_t(blockIdx.x) * 64;
  const int c0 = blockIdx.y * 64;
  if (r0 >= T_pad) {   // uniform over the workgroup
    if (blockIdx.y == 0) loss_reduce<256>(term, flag, nact[0], loss, clip_frac);
    return;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int u = threadIdx.x + k * 256;
    const int rr = u >> 3, c8 = (u & 7) * 8;
    const int64_t r = r0 + rr;
    const int c = c0 + c8;
    u32x4_t v = {0u, 0u, 0u, 0u};
    if (c < C) {
      v = *reinterpret_cast<const u32x4_t*>(in + r * C + c);
      const float f = scale[r];
      float x[8];
      unpack8(v, x);
      v.x = pack_bf16x2(x[0] * f, x[1] * f);
      v.y = pack_bf16x2(x[2] * f, x[3] * f);
      v.z = pack_bf16x2(x[4] * f, x[5] * f);
      v.w = pack_bf16x2(x[6] * f, x[7] * f);
    }
    tile[rr][c8 / 2 + 0] = v.x;
    tile[rr][c8 / 2 + 1] = v.y;
    tile[rr][c8 / 2 + 2] = v.z;
    tile[rr][c8 / 2 + 3] = v.w;
  }
  __syncthreads();
  uint16_t* slab = out + slab_offset(T_pad / 64, c0 / kTile, blockIdx.x) + c0 % kTile * 64;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int u = threadIdx.x + k * 256;
    const int cc = u >> 3, q = u & 7;   // column cc, K positions 8 q .. 8 q + 7
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t lo = tile[8 * q + 2 * e][cc >> 1], hi = tile[8 * q + 2 * e + 1][cc >> 1];
      w[e] = (cc & 1) ? ((lo >> 16) | (hi & 0xffff0000u)) : ((lo & 0xffffu) | (hi << 16));
    }
    const u32x4_t v = {w[0], w[1], w[2], w[3]};
    *reinterpret_cast<u32x4_t*>(slab + cc * 64 + 8 * q) = v;
  }
}

// ------------------------------------------------------------------------------------------
// backward: dz tiles, whole vocabulary
// ------------------------------------------------------------------------------------------
// z^T tile rows = vocab [m0, m0 + 256), columns = compacted tokens.  The bf16 gradient leaves in
// the two layouts the next two contractions read, both K-slabs in fragment order (frag_order_offset): dz tokens x
// vocabulary, and dzT vocabulary x tokens; entries outside the vocabulary or the candidate tokens are zero.
// ENT: rows also carry the entropy-bonus term, dz = pi (ac z + bc) + gc onehot; otherwise ac = 0
// and the scale is the per-token constant bc = -g.
// The kernel is the recompute mode of the backward pass (see FusedTerms): with force == 0 it
// leaves at once unless the forward pass raised nact[2].
template <bool ENT>
__global__ __launch_bounds__(kGemmNT, 2) void k_fused_dz(
    const uint16_t* __restrict__ W, const uint16_t* __restrict__ Hc, int V, int H,
    int tiles_v, int64_t T_pad, int V_ld, int force, const int32_t* __restrict__ nact,
    const float* __restrict__ gc, const float* __restrict__ lsec, const int32_t* __restrict__ yc,
    const float* __restrict__ ac, const float* __restrict__ bc, uint16_t* __restrict__ dz,
    uint16_t* __restrict__ dzT) {
  extern __shared__ __align__(16) uint16_t smem[];
  if (!force && nact[2] == 0) return;   // uniform over the launch
  // tile order over the candidates' token tiles only (see k_fused_stats)
  const int tiles_t_act = nact[1] / kTile, n_cand = nact[0];
  const int n_tiles = tiles_v * tiles_t_act;
  WavePos wp = wave_pos<true>();
  const int wm = wp.wm, wn = wp.wn;
  GemmStream<true, false, false, true> stream(H, kDK, H, kDK, H);
  auto source = [&](int tv, int tt) {
    return TileSrc{W, Hc, (int64_t(V) * H) * 2, (int64_t(n_cand) * H) * 2, uint32_t(int64_t(tv) * kTile * H * 2),
                   uint32_t(int64_t(tt) * kTile * H * 2), (H + kDK - 1) / kDK};
  };
  int pid = blockIdx.x, tv, tt;
  bool more = tile_of_step(pid, tiles_v, tiles_t_act, 0, n_tiles, tv, tt), stored = false;
  if (!more) return;
  TileSrc src = source(tv, tt);
  stream.start(src, smem);
  while (more) {
    const int m0 = tv * kTile, n0 = tt * kTile;
    wp.active = n0 + wn * 64 < n_cand;
    wp.warm_a = warm_share(tt, tiles_t_act);
    wp.warm_b = warm_share(tv, tiles_v);
    wp.warm_from = forward_warm_from(tiles_t_act);
    pid += gridDim.x;
    more = tile_of_step(pid, tiles_v, tiles_t_act, 0, n_tiles, tv, tt);
    const TileSrc next = more ? source(tv, tt) : no_tile(src);
    Acc acc;
    stream.run<kTileStores>(src, next, wp, stored, smem, acc);
    src = next;
    stored = n0 + wn * 64 < n_cand;   // uniform over the wave: nobody reads 64 columns without a candidate
    if (!stored) continue;

    const int lane = opaque(threadIdx.x & 63);
    // dz for this lane's columns, packed to bf16 pairs: pk[nb][mb] = four consecutive rows
    uint32_t pk[kNB][kMB][2];
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) {
      const int64_t t = n0 + acc_col(wn, nb, lane);
      const float g = gc[t], ng = bc[t];   // bc = -g without the entropy bonus
      const float a = ENT ? ac[t] : 0.f;
      const float c = -lsec[t] * kLog2e;
      const int yrel = yc[t];        // vocabulary row of the sampled token (-1 on padding columns)
      // Almost every wave holds neither a sampled token's row nor rows past the vocabulary: that
      // case (uniform over the wave) runs without the two per-element tests.
      const bool plain = (m0 + kTile <= V) && !__any(unsigned(yrel - m0 - wm * 128) < 128u);
#pragma unroll
      for (int mb = 0; mb < kMB; ++mb) {
        float d[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float z = acc[mb][nb][j];
          d[j] = (ENT ? fmaf(a, z, ng) : ng) * exp2_fast(fmaf(z, kLog2e, c));
        }
        if (!plain) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int row = m0 + acc_row(wm, mb, j, lane);
            if (row == yrel) d[j] += g;
            if (row >= V) d[j] = 0.f;
          }
        }
        pk[nb][mb][0] = pack_bf16x2(d[0], d[1]);
        pk[nb][mb][1] = pack_bf16x2(d[2], d[3]);
      }
    }
    store_tile_both_layouts(pk, wp, lane, m0, n0, T_pad, V_ld, dz, dzT);
  }
  end_of_walk();
}

// ------------------------------------------------------------------------------------------
// backward: the two gradient GEMMs
// ------------------------------------------------------------------------------------------
// dh_part[s][t][h] = sum_{k in split s} X[t][k] W[k][h], X = the stored exponentials P (or dz itself on the recompute
// route)     M = candidate tokens, N = H, K = vocabulary (padded)
// The weight is read as the caller holds it, [V][H], and turned by the transposing LDS read.  (A copy of it in K-slabs costs a
// pass over the weight per call, 170 us at H = 1536 and 430 at 3584 with V = 152 K; with two stages of 64 the contraction gained
// at most 2 % by it.)
__device__ __forceinline__ void dh_tile(int block, uint16_t* smem, const uint16_t* __restrict__ dz, const uint16_t* __restrict__ W,
                                        int V, int vK, int H, int tiles_h, const int32_t* __restrict__ nact,
                                        float* __restrict__ dh_part) {
  const int n_pad = nact[1], n_cand = nact[0];
  const int tiles_t = n_pad / kTile;
  const int nslices = vK / kDK;
  const int S = nact[3];
  const int base = tiles_t * tiles_h, n = base * S;
  if (block >= n) return;   // uniform over the workgroup
  const int per = (nslices + S - 1) / S;
  WavePos wp = wave_pos<false>();
  const int wm = wp.wm, wn = wp.wn;
  const GemmRing ring(H, smem);
  auto source = [&](int split, int tt, int th) {
    const int k_begin = min(vK, split * per * kDK);
    const int k_len = max(0, min(vK, (split + 1) * per * kDK) - k_begin);
    RingSrc t;
    t.a_base = dz + slab_offset(nslices, tt, k_begin / kDK);
    t.a_bytes = uint32_t(k_len) * (kTile * 2);
    t.a_rows = n_cand - tt * kTile;   // blocks of rows without a candidate are not requested
    // weight rows past the vocabulary (the split may start there) lie past the operand's bytes and read as zeros
    t.b_base = W + int64_t(min(k_begin, V)) * H;
    t.b_bytes = uint32_t(max(min(V - k_begin, k_len), 0)) * uint32_t(H) * 2;
    t.b = uint32_t(th * kTile * 2);
    t.nk = max(k_len / kStepK, 4);    // steps past a short split's end are zeros
    return t;
  };
  // per-XCD contiguous order, split-major: the workgroups resident on one XCD work on the same
  // K range of neighbouring tiles and share their operand slices in that XCD's L2
  const int npid = xcd_regroup(block, n);
  const int split = npid / base;
  int tt, th;
  tile_of_index(npid % base, tiles_t, tiles_h, tt, th);
  const int m0 = tt * kTile, n0 = th * kTile;
  wp.active = m0 + wm * 128 < n_cand && n0 + wn * 64 < H;
  Acc acc;
  ring.run(source(split, tt, th), wp, smem, acc);
  if (!wp.active) return;   // padding rows of the partials are not read, columns past H do not exist
  const int lane = threadIdx.x & 63;
  float* const out = dh_part + int64_t(split) * n_pad * H;
#pragma unroll
  for (int mb = 0; mb < kMB; ++mb) {
    float* row = out + int64_t(m0 + acc_row_swapped(wm, mb, lane)) * H;
#pragma unroll
    for (int nb = 0; nb < kNB; ++nb) {
      const int col = n0 + acc_col_swapped(wn, nb, lane);   // four columns; H is a multiple of 8
      if (col < H) *reinterpret_cast<f32x4_t*>(row + col) = acc[mb][nb];
    }
  }
}

__global__ __launch_bounds__(kGemmNT, 2) void k_gemm_dh(
    const uint16_t* __restrict__ dz, const uint16_t* __restrict__ W, int V, int vK, int H, int tiles_h,
    const int32_t* __restrict__ nact, float* __restrict__ dh_part) {
  extern __shared__ __align__(16) uint16_t smem[];
  dh_tile(blockIdx.x, smem, dz, W, V, vK, H, tiles_h, nact, dh_part);
}

// Calls of at least so many rows get a workgroup per tile, smaller ones a workgroup per CU that walks the tiles: walking pays for
// a tile's start and drain, which counts where the contraction is short, and loses 0.5-3 % of a call where it is long.
// Walking / per tile, whole calls: every row a candidate, H = 1536, V = 151936: 64 slices 4881 / 4895 us (bf16), 128 9854 / 9838, 160
// 12799 / 12703, 250 20215 / 19900 (added to dweight 20523 / 20054), 330 27545 / 27152; H = 2048 128 slices 10696 / 10587; H = 3584
// 96 slices 16593 / 16610, 375 68040 / 66109.  62 % of the rows: 8192 rows 7403 / 7408, 10240 9600 / 9573, 16384 14568 / 14541.  The
// host knows the rows, not how many are candidates.
constexpr int64_t kDwTileRows = 8192;

// dW[m][h] = sum_t XT[m][t] hTc[h][t], hTc = the candidates' hidden rows times their scale     M = V, N = H, K = candidate tokens (padded)
// Workgroup `block` of `blocks`.  parts > 1: dW is [parts][V][H].
template <bool OUT_BF16, bool ACC>
__device__ __forceinline__ void dw_tiles(int block, int blocks, uint16_t* smem, const uint16_t* __restrict__ dzT,
                                         const uint16_t* __restrict__ hTc, int V, int H, int tile0, int n_tiles, int tiles_v, int tiles_h,
                                         int64_t T_pad, const int32_t* __restrict__ nact, int vec, int parts, void* dW) {
  // the contraction ends with the slice of the last candidate, not with its tile: the positions behind it are zeros
  // (whole calls at H = 1536, V = 151936: 600 tokens 949 -> 905 us, 1100 tokens 1376 -> 1357, 16384 tokens -0.4 %)
  const int slices = (nact[0] + kDK - 1) / kDK;
  // parts are further rows of tiles, part by part; tv counts through them
  const int per = (slices + parts - 1) / parts;
  WavePos wp = wave_pos<true>();
  const int wm = wp.wm, wn = wp.wn;
  GemmStream<true, true, true, false> stream(kDK, kSlabElems, kDK, kSlabElems, 0);
  auto source = [&](int tv, int th) {
    const bool any = th * kTile + stream.wave * 32 < H;   // of the 32 columns that the wave requests
    const int part = parts > 1 ? tv / tiles_v : 0, begin = part * per, n = max(min(per, slices - begin), 0);
    if (parts > 1) tv -= part * tiles_v;
    return TileSrc{dzT + slab_offset(T_pad / 64, tv, begin), hTc + slab_offset(T_pad / 64, th, begin), int64_t(n) * kSlabElems * 2,
                   any ? int64_t(n) * kSlabElems * 2 : 0, 0u, 0u, max(n, 1)};   // no candidates: one slice of nothing
  };
  // accumulate (uniform): the tile is added to what the caller's buffer holds (gradient accumulation over
  // micro-batches).  vec (uniform): that buffer is 16-byte aligned, as every allocation is.  Plain stores: an
  // instruction writes 64 bytes per row and L2 joins the two halves of a line; non-temporal ones leave it in
  // halves (1.4 times the gradient's bytes written, 312 against 287 us with 600 tokens at H = 1536,
  // V = 151936 in bf16 while the contraction took whole token tiles - 223 us since it ends earlier -, 1690 against
  // 1660 us per 1536 tiles with 16384 in fp32).
  constexpr int kDT = OUT_BF16 ? kBF16 : kF32;
  int pid = block, tv, th;
  bool more = tile_of_step(pid, parts * tiles_v, tiles_h, tile0, n_tiles, tv, th), stored = false;
  if (!more) return;
  TileSrc src = source(tv, th);
  stream.start(src, smem);
  while (more) {
    const int part = parts > 1 ? tv / tiles_v : 0;
    const int m0 = (tv - part * tiles_v) * kTile, n0 = th * kTile;
    wp.active = n0 + wn * 64 < H;
    wp.warm_a = warm_share(th, tiles_h);
    wp.warm_b = warm_share(tv, tiles_v);
    wp.warm_from = kWarmSlices;
    pid += blocks;
    more = tile_of_step(pid, parts * tiles_v, tiles_h, tile0, n_tiles, tv, th);
    const TileSrc next = more ? source(tv, th) : no_tile(src);
    Acc acc;
    stream.template run<OUT_BF16 ? kMB * kNB / 2 : kMB * kNB>(src, next, wp, stored, smem, acc);
    src = next;
    stored = vec && m0 + kTile <= V && n0 + kTile <= H;   // then every store below is issued
    const int lane = opaque(threadIdx.x & 63);
#pragma unroll
    for (int mb = 0; mb < kMB; ++mb) {
      const int row = m0 + acc_row_swapped(wm, mb, lane);
      const int64_t row_off = (int64_t(part) * V + row) * H;
      const bool row_in = row < V;
      if (!vec) {
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) {
          const int col = n0 + acc_col_swapped(wn, nb, lane);
          if (!row_in || col >= H) continue;
#pragma unroll
          for (int i = 0; i < 4; ++i)
            store_elt<kDT>(dW, row_off + col + i, acc[mb][nb][i] + (ACC ? load_elt<kDT>(dW, row_off + col + i) : 0.f));
        }
      } else if constexpr (OUT_BF16) {
        if constexpr (ACC) {
#pragma unroll
          for (int nb = 0; nb < kNB; ++nb) {
            const int col = n0 + acc_col_swapped(wn, nb, lane);
            if (!row_in || col >= H) continue;
            const uint64_t old = __builtin_nontemporal_load(reinterpret_cast<const uint64_t*>(reinterpret_cast<uint16_t*>(dW) + row_off + col));
            const uint32_t lo = uint32_t(old), hi = uint32_t(old >> 32);
            acc[mb][nb] += f32x4_t{bf16_lo(lo), bf16_hi(lo), bf16_lo(hi), bf16_hi(hi)};
          }
        }
        // Two neighbouring blocks: the odd 16-lane rows of the first change places with the even ones of the
        // second, so that every lane holds eight consecutive columns and an instruction writes 64 contiguous
        // bytes per vocabulary row.  (8-byte stores, 32 contiguous bytes: 454 us where these take 312, at
        // 600 tokens.)
#pragma unroll
        for (int nb = 0; nb < kNB; nb += 2) {
          const auto lo = __builtin_amdgcn_permlane16_swap(pack_bf16x2(acc[mb][nb].x, acc[mb][nb].y),
                                                           pack_bf16x2(acc[mb][nb + 1].x, acc[mb][nb + 1].y), false, false);
          const auto hi = __builtin_amdgcn_permlane16_swap(pack_bf16x2(acc[mb][nb].z, acc[mb][nb].w),
                                                           pack_bf16x2(acc[mb][nb + 1].z, acc[mb][nb + 1].w), false, false);
          const int group = lane >> 4;
          const int col = n0 + wn * 64 + (nb + (group & 1)) * 16 + (group >> 1) * 8;
          if (row_in && col < H)
            *reinterpret_cast<u32x4_t*>(reinterpret_cast<uint16_t*>(dW) + row_off + col) = u32x4_t{lo[0], hi[0], lo[1], hi[1]};
        }
      } else {
#pragma unroll
        for (int nb = 0; nb < kNB; ++nb) {
          const int col = n0 + acc_col_swapped(wn, nb, lane);
          if (!row_in || col >= H) continue;
          f32x4_t* const p = reinterpret_cast<f32x4_t*>(reinterpret_cast<float*>(dW) + row_off + col);
          if constexpr (ACC) acc[mb][nb] += __builtin_nontemporal_load(p);
          *p = acc[mb][nb];
        }
      }
    }
  }
  end_of_walk();
}

template <bool OUT_BF16, bool ACC>
__global__ __launch_bounds__(kGemmNT, 2) void k_gemm_dw(
    const uint16_t* __restrict__ dzT, const uint16_t* __restrict__ hTc, int V, int H, int tile0, int n_tiles, int tiles_v, int tiles_h,
    int64_t T_pad, const int32_t* __restrict__ nact, int vec, void* dW) {
  extern __shared__ __align__(16) uint16_t smem[];
  dw_tiles<OUT_BF16, ACC>(blockIdx.x, gridDim.x, smem, dzT, hTc, V, H, tile0, n_tiles, tiles_v, tiles_h, T_pad, nact, vec, 1, dW);
}

// Both contractions in one launch: the workgroups that walk dweight's tiles, then (from dw_blocks on, a multiple of 8) dhidden's, which
// take the CUs that the former leave idle or are through with.  For H up to 256, where dhidden has at most 64 splits of a few tiles, and
// for gradients of up to a tile per CU; calls of kDwTileRows rows and more fill the chip with either, unless the gradient has few
// tiles (up to kDwSplitTiles; its range in one part, two launches / one: H = 64, V = 4000 20000 rows 397 / 379 us, H = 896, V = 8000 801 / 727).  Whole calls, two launches / one: H = 208,
// V = 152064 144 rows 133.7 / 122.7 us, 500 248 / 217, 2000 659 / 601, 6000 1593 / 1542; H = 256, V = 60000 500 120.6 / 117.9, 4000 470 / 444; H = 360,
// V = 4249 1080 rows 83.9 / 70.9; H = 896, V = 5504 1001 103.5 / 97.3; H = 2048, V = 6678 240 108.5 / 107.1; 75 calls drawn over
// the rule's range (128 to 8192 rows, H to 2560, V to 150 K) 0.99 to 1.23 times as fast, 1.09 in the median.  Where both fill the chip it is a matter of
// how their last rounds fall: H = 896, V = 33846 500 rows 172.5 / 174.3, 4000 693 / 659; H = 640, V = 30000 4000 451 / 460; H = 3584, V = 32000 300 272 / 280.
template <bool OUT_BF16, bool ACC, bool SPLIT>
__global__ __launch_bounds__(kGemmNT, 2) void k_gemm_grads(
    const uint16_t* __restrict__ dz, const uint16_t* __restrict__ W, int vK, float* dh_part, int dw_blocks,
    const uint16_t* __restrict__ dzT, const uint16_t* __restrict__ hTc, int V, int H, int n_tiles, int tiles_v, int tiles_h,
    int64_t T_pad, const int32_t* __restrict__ nact, int vec, void* dW) {
  extern __shared__ __align__(16) uint16_t smem[];
  const int parts = SPLIT ? nact[4] : 1;   // uniform over the launch
  if (int(blockIdx.x) < dw_blocks && parts > 1)
    dw_tiles<false, false>(blockIdx.x, dw_blocks, smem, dzT, hTc, V, H, 0, parts * n_tiles, tiles_v, tiles_h, T_pad, nact, 1, parts,
                           dh_part + dw_part_offset(nact, H));
  else if (int(blockIdx.x) < dw_blocks)
    dw_tiles<OUT_BF16, ACC>(blockIdx.x, dw_blocks, smem, dzT, hTc, V, H, 0, n_tiles, tiles_v, tiles_h, T_pad, nact, vec, 1, dW);
  else
    dh_tile(int(blockIdx.x) - dw_blocks, smem, dz, W, V, vK, H, tiles_h, nact, dh_part);
}

// dweight from its parts: [parts][V][H] fp32, added up in order, eight entries (n of them) a thread.
template <bool OUT_BF16, bool ACC>
__device__ __forceinline__ void sum_dw(int64_t block, int parts, const float* __restrict__ part, int64_t n, int vec, void* dW) {
  constexpr int kDT = OUT_BF16 ? kBF16 : kF32;
  const int64_t at = (block * 256 + threadIdx.x) * 8;
  if (at >= n) return;
  f32x4_t lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll 4
  for (int p = 0; p < parts; ++p) {
    const f32x4_t* const src = reinterpret_cast<const f32x4_t*>(part + p * n + at);
    lo += src[0];
    hi += src[1];
  }
  float x[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
  if (!vec) {
#pragma unroll
    for (int e = 0; e < 8; ++e) store_elt<kDT>(dW, at + e, x[e] + (ACC ? load_elt<kDT>(dW, at + e) : 0.f));
    return;
  }
  u32x4_t* const out = reinterpret_cast<u32x4_t*>(reinterpret_cast<char*>(dW) + at * Storage<kDT>::kBytes);
  if constexpr (OUT_BF16) {
    if constexpr (ACC) {
      float old[8];
      unpack8(out[0], old);
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] += old[e];
    }
    out[0] = pack_vec<kBF16>(x);
  } else {
    if constexpr (ACC) {
      lo += *reinterpret_cast<const f32x4_t*>(out);
      hi += *reinterpret_cast<const f32x4_t*>(out + 1);
    }
    *reinterpret_cast<f32x4_t*>(out) = lo;
    *reinterpret_cast<f32x4_t*>(out + 1) = hi;
  }
}

// dhidden[t] = bf16(scale[pos[t]] * sum over the split-K partials of row pos[t]) or +0.  One workgroup per
// row; the partials are summed in split order, so the result does not depend on scheduling.
__device__ __forceinline__ void scatter_dh(int64_t t, const float* __restrict__ dh_part, const int32_t* __restrict__ pos,
                                           const int32_t* __restrict__ nact, int H, const float* __restrict__ scale,
                                           uint16_t* __restrict__ dhidden) {
  const int j = pos[t];
  uint16_t* out = dhidden + t * H;   // H % 8 == 0 and a 16-byte aligned base: rows are whole 16-byte vectors
  const float f = j < 0 ? 0.f : scale[j];
  if (f == 0.f) {   // no gradient row, or one whose token was clipped
    for (int k = threadIdx.x * 8; k < H; k += 256 * 8) *reinterpret_cast<u32x4_t*>(out + k) = u32x4_t{0u, 0u, 0u, 0u};
    return;
  }
  const int n_pad = nact[1];
  const int S = nact[3];
  for (int k = threadIdx.x * 4; k < H; k += 256 * 4) {
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    const float* src = dh_part + int64_t(j) * H + k;
    const int64_t step = int64_t(n_pad) * H;
    int s = 0;
    auto add = [&](auto count) {   // so many loads in flight, added in split order
      constexpr int N = decltype(count)::value;
      f32x4_t v[N];
#pragma unroll
      for (int u = 0; u < N; ++u) v[u] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t*>(src + (s + u) * step));
#pragma unroll
      for (int u = 0; u < N; ++u) acc += v[u];
      s += N;
    };
    while (s + 12 <= S) add(std::integral_constant<int, 12>{});
    if (s + 8 <= S) add(std::integral_constant<int, 8>{});
    if (s + 4 <= S) add(std::integral_constant<int, 4>{});
    if (s + 2 <= S) add(std::integral_constant<int, 2>{});
    if (s < S) add(std::integral_constant<int, 1>{});
    uint2 o;
    o.x = pack_bf16x2(acc.x * f, acc.y * f);
    o.y = pack_bf16x2(acc.z * f, acc.w * f);
    *reinterpret_cast<uint2*>(out + k) = o;
  }
}

__global__ __launch_bounds__(256) void k_scatter_dh(const float* __restrict__ dh_part, const int32_t* __restrict__ pos,
                                                    const int32_t* __restrict__ nact, int H,
                                                    const float* __restrict__ scale, uint16_t* __restrict__ dhidden) {
  scatter_dh(blockIdx.x, dh_part, pos, nact, H, scale, dhidden);
}

// The same, and dweight from its parts in the workgroups behind the first T, which leave at once where it is in one part.
template <bool OUT_BF16, bool ACC>
__global__ __launch_bounds__(256) void k_scatter_and_sum(const float* __restrict__ dh_part, const int32_t* __restrict__ pos,
                                                         const int32_t* __restrict__ nact, int H, const float* __restrict__ scale,
                                                         uint16_t* __restrict__ dhidden, unsigned T, int64_t n, int vec, void* dW) {
  if (blockIdx.x < T)
    scatter_dh(blockIdx.x, dh_part, pos, nact, H, scale, dhidden);
  else if (nact[4] > 1)
    sum_dw<OUT_BF16, ACC>(blockIdx.x - T, nact[4], dh_part + dw_part_offset(nact, H), n, vec, dW);
}

static aero_status set_lds(const void* fn) {
  return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, int(kGemmLdsBytes)) == hipSuccess
             ? AERO_OK : AERO_ERR_HIP;
}

}  // namespace aero

extern "C" aero_status aero_lmhead_logprob_fused(
    const void* hidden, const void* weight, int64_t T, int32_t H, int32_t V, const int32_t* targets,
    float* logprob, float* entropy, float* lse, const float* old_logprob, const int32_t* token_rollout,
    const float* adv, const float* weight_rollout, int32_t R, float eps_lo, float eps_hi, float grad_scale,
    float entropy_coef, float kl_coef, const float* ref_logprob, float* loss, float* clip_frac, void* dhidden,
    void* dweight, int32_t dweight_dtype, int32_t* err_flag, void* workspace, size_t workspace_bytes, void* stream) {
  using namespace aero;
  if (!(entropy_coef == entropy_coef) || !(kl_coef == kl_coef)) return AERO_ERR_SHAPE;   // NaN coefficient
  if (old_logprob && kl_coef != 0.f && T > 0 && !ref_logprob) return AERO_ERR_NULL;
  if (T < 0 || T > 0x7fffff00LL || V < 1 || V > (1 << 24) || H < 8 || H % 8 != 0 || H > (1 << 20) || R < 0)
    return AERO_ERR_SHAPE;
  const bool bwd = old_logprob != nullptr;
  const int accumulate = (dweight_dtype & AERO_DW_ACCUMULATE) ? 1 : 0;
  dweight_dtype &= ~AERO_DW_ACCUMULATE;
  if (bwd && dweight_dtype != AERO_F32 && dweight_dtype != AERO_BF16) return AERO_ERR_DTYPE;
  if (!weight) return AERO_ERR_NULL;
  if (T > 0 && (!hidden || !targets || !logprob || !lse)) return AERO_ERR_NULL;
  if (bwd && (!loss || !dweight || (T > 0 && (!token_rollout || !adv || !weight_rollout || !dhidden))))
    return AERO_ERR_NULL;
  if (reinterpret_cast<uintptr_t>(hidden) % 16 || reinterpret_cast<uintptr_t>(weight) % 16) return AERO_ERR_ALIGN;
  if (bwd && reinterpret_cast<uintptr_t>(dhidden) % 16) return AERO_ERR_ALIGN;   // rows are written as 16-byte vectors
  const FusedPlan p = make_plan(T, V, H);
  // operands are addressed with 32-bit byte offsets: a tile's run of slabs, the hidden rows and the weight must stay below 4 GiB
  constexpr size_t kOperandLimit = size_t(1) << 32;
  if (size_t(p.H_pad) * size_t(p.T_pad) * 2 >= kOperandLimit || size_t(p.T_pad) * kTile * 2 >= kOperandLimit ||
      size_t(V) * size_t(H) * 2 >= kOperandLimit)
    return AERO_ERR_SHAPE;
  {  // the split-K dhidden contraction must find a split count whose K ranges stay below that limit
    const int64_t rows = p.T_pad > p.H_pad ? p.T_pad : int64_t(p.H_pad);
    const int64_t s_min = (int64_t(p.V_ld) * rows * 2 + kOperandBytes - 1) / kOperandBytes;
    if (s_min + 1 > 64 || rows * (s_min + 1) >= (int64_t(1) << 25)) return AERO_ERR_SHAPE;
  }
  // one workgroup per 256 x 256 tile: the tile count must fit a launch grid
  if (int64_t(p.tiles_v) * (p.T_pad / kTile) >= (int64_t(1) << 31) - 64) return AERO_ERR_SHAPE;   // grids are rounded up to 64
  if (!workspace || reinterpret_cast<uintptr_t>(workspace) % kWsAlign || workspace_bytes < p.total)
    return AERO_ERR_WORKSPACE;
  hipStream_t s = as_stream(stream);
  char* ws = reinterpret_cast<char*>(workspace);
  const uint16_t* Wp = reinterpret_cast<const uint16_t*>(weight);
  const uint16_t* Hp = reinterpret_cast<const uint16_t*>(hidden);
  float* part_m = reinterpret_cast<float*>(ws + p.off_part);
  float* part_s = part_m + size_t(p.tiles_v) * p.T_pad;
  float* part_sz = part_s + size_t(p.tiles_v) * p.T_pad;
  const int tiles_t = int(p.T_pad / kTile);
  const int tiles_h = (H + kTile - 1) / kTile;
  const int grid_dh = dh_grid(p.T_pad, H, p.V_ld);
  // contractions: one workgroup per CU walks the tiles (exceptions: kDwTileRows, kForwardTileSlices); a multiple of 8 keeps a walk on its XCD
  const int cus = compute_units() / 8 * 8 > 0 ? compute_units() / 8 * 8 : 8;
  auto walkers = [&](int n) { return dim3(unsigned(n < cus ? n : cus)); };
  auto forward_grid = [&](int n) { return (H + kDK - 1) / kDK < kForwardTileSlices ? walkers(xcd_grid(n)) : dim3(unsigned(xcd_grid(n))); };
  const int64_t rows_max = p.T_pad > p.H_pad ? p.T_pad : int64_t(p.H_pad);

  // raising the dynamic-LDS limit is per function; done once per process, safely from any thread
  static std::once_flag attr_once;
  static aero_status attr_rc = AERO_OK;
  std::call_once(attr_once, [] {
    if (set_lds(reinterpret_cast<const void*>(k_fused_stats<false>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_fused_stats<true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_fused_dz<false>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_fused_dz<true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_dh)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<true, true, true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<true, true, false>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<true, false, true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<true, false, false>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<false, true, true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<false, true, false>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<false, false, true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_grads<false, false, false>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_dw<true, true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_dw<true, false>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_dw<false, true>)) != AERO_OK ||
        set_lds(reinterpret_cast<const void*>(k_gemm_dw<false, false>)) != AERO_OK)
      attr_rc = AERO_ERR_HIP;
  });
  if (attr_rc != AERO_OK) return attr_rc;

  // ---- forward ----
  int32_t* fidx = reinterpret_cast<int32_t*>(ws + p.off_fidx);
  int32_t* nf = reinterpret_cast<int32_t*>(ws + p.off_nf);
  int32_t* pos = reinterpret_cast<int32_t*>(ws + p.off_pos);
  int32_t* nact = reinterpret_cast<int32_t*>(ws + p.off_nact);
  float* zy = reinterpret_cast<float*>(ws + p.off_zy);
  uint16_t* hf = reinterpret_cast<uint16_t*>(ws + p.off_hc);   // rows with a target, candidates first
  uint16_t* dz = reinterpret_cast<uint16_t*>(ws + p.off_dz);
  uint16_t* dzT = reinterpret_cast<uint16_t*>(ws + p.off_dzT);
  const bool ent = bwd && entropy_coef != 0.f;
  // rows with an entropy term are not a multiple of exp(z - zy): their gradient is formed by recomputing z
  const bool stored = bwd && !ent;
  FusedTerms terms{};
  if (bwd)
    terms = FusedTerms{targets, token_rollout, old_logprob, adv, weight_rollout, ref_logprob,
                       LossHyper{eps_lo, eps_hi, grad_scale, entropy_coef, kl_coef}, nact, p.T_pad, p.V_ld, stored ? 0 : 1,
                       reinterpret_cast<float*>(ws + p.off_term), reinterpret_cast<int32_t*>(ws + p.off_flag),
                       reinterpret_cast<float*>(ws + p.off_gc), reinterpret_cast<float*>(ws + p.off_lsec),
                       reinterpret_cast<int32_t*>(ws + p.off_yc), reinterpret_cast<float*>(ws + p.off_ac),
                       reinterpret_cast<float*>(ws + p.off_bc), reinterpret_cast<float*>(ws + p.off_scale), dz, dzT};
  const int total = p.tiles_v * tiles_h;
  DwSplit split{1, total, V, dh_part_rows(p.T_pad, H, p.V_ld)};
  if (bwd && total <= kDwSplitTiles && dw_split_pays(total, (T + kDK - 1) / kDK))   // if every row is a candidate
    split.most = std::max(std::min(cus / total, kDwSplitMax), 1);
  const auto compact = T <= 2048 ? k_compact_valid<1> : k_compact_valid<4>;   // steps of 1024 rows at a time
  if (T > 0) {
    hipLaunchKernelGGL(compact, dim3(1), dim3(1024), 0, s, targets, T, p.T_pad, V,
                       bwd ? token_rollout : nullptr, adv, weight_rollout, R, (ent || kl_coef != 0.f) ? 1 : 0, fidx, nf,
                       bwd ? pos : nullptr, bwd ? nact : nullptr, logprob, entropy, lse, err_flag, tiles_h, grid_dh,
                       p.V_ld / kDK, rows_max, split);
    hipLaunchKernelGGL(k_gather_rows, dim3(unsigned(p.T_pad / 4)), dim3(256), 0, s, Hp, Wp, H, fidx, targets, hf, zy);
    {
      const int n = p.tiles_v * tiles_t;
      if (stored)
        hipLaunchKernelGGL(k_fused_stats<true>, forward_grid(n), dim3(kGemmNT), kGemmLdsBytes, s, Wp, hf,
                           V, H, p.tiles_v, p.T_pad, nf, part_m, part_s, part_sz, zy, p.V_ld, nact, dz, dzT);
      else
        hipLaunchKernelGGL(k_fused_stats<false>, forward_grid(n), dim3(kGemmNT), kGemmLdsBytes, s, Wp, hf,
                           V, H, p.tiles_v, p.T_pad, nf, part_m, part_s, part_sz, zy, p.V_ld, nact, dz, dzT);
    }
    if (p.T_pad <= kFewRows)
      hipLaunchKernelGGL(k_fused_rows<16>, dim3(unsigned(p.T_pad / 16)), dim3(kRowsNT), 0, s, p.tiles_v, p.T_pad, fidx, nf,
                         part_m, part_s, part_sz, zy, logprob, entropy, lse, terms);
    else
      hipLaunchKernelGGL(k_fused_rows<64>, dim3(unsigned(p.T_pad / 64)), dim3(kRowsNT), 0, s, p.tiles_v, p.T_pad, fidx, nf,
                         part_m, part_s, part_sz, zy, logprob, entropy, lse, terms);
  }
  if (!bwd) return launch_status();

  // ---- loss, operand copy ----
  uint16_t* hTc = reinterpret_cast<uint16_t*>(ws + p.off_hTc);
  float* dh_acc = reinterpret_cast<float*>(ws + p.off_dhacc);
  if (T == 0) {   // no forward kernel ran: an empty candidate set for the kernels below
    hipLaunchKernelGGL(compact, dim3(1), dim3(1024), 0, s, targets, T, p.T_pad, V, token_rollout, adv,
                       weight_rollout, R, 0, fidx, nf, pos, nact, logprob, entropy, lse, err_flag, tiles_h, grid_dh,
                       p.V_ld / kDK, rows_max, split);
    hipLaunchKernelGGL(k_fused_rows<16>, dim3(unsigned(p.T_pad / 16)), dim3(kRowsNT), 0, s, p.tiles_v, p.T_pad, fidx, nf,
                       part_m, part_s, part_sz, zy, logprob, entropy, lse, terms);
  }
  if (T > 0) {   // recompute mode only (the kernel leaves at once otherwise)
    const int n = p.tiles_v * tiles_t;
    if (ent)
      hipLaunchKernelGGL(k_fused_dz<true>, forward_grid(n), dim3(kGemmNT), kGemmLdsBytes, s, Wp, hf, V,
                         H, p.tiles_v, p.T_pad, p.V_ld, terms.force_recompute, nact, terms.gc, terms.lsec, terms.yc, terms.ac,
                         terms.bc, dz, dzT);
    else
      hipLaunchKernelGGL(k_fused_dz<false>, forward_grid(n), dim3(kGemmNT), kGemmLdsBytes, s, Wp, hf, V,
                         H, p.tiles_v, p.T_pad, p.V_ld, terms.force_recompute, nact, terms.gc, terms.lsec, terms.yc, terms.ac,
                         terms.bc, dz, dzT);
  }
  hipLaunchKernelGGL(k_hidden_and_loss, dim3(unsigned(p.T_pad / 64 + 1), unsigned(p.H_pad / 64)), dim3(256), 0, s, hf, p.T_pad, H,
                     p.H_pad, hTc, terms.scale, terms.term, terms.flag, nact, loss, clip_frac);

  // ---- the two gradient contractions over the whole vocabulary ----
  // dz columns [V, V_ld) are zero, weight rows past V read as zeros: the contraction runs over the padded vocabulary
  const int vec_dw = reinterpret_cast<uintptr_t>(dweight) % 16 == 0;   // rows are multiples of 16 bytes
  const bool dw_bf16 = dweight_dtype == AERO_BF16;
  uint16_t* const dh = reinterpret_cast<uint16_t*>(dhidden);
  const bool together = total <= std::min(kDwSplitTiles, cus) || (p.T_pad < kDwTileRows && (tiles_h == 1 || total <= cus));
  if (T > 0 && together) {   // see k_gemm_grads
    auto launch = [&](auto out, auto acc) {
      constexpr bool OUT = decltype(out)::value, ACC = decltype(acc)::value;
      const int dw_blocks = int(walkers(xcd_grid(split.most * total)).x);
      const auto grads = split.most > 1 ? k_gemm_grads<OUT, ACC, true> : k_gemm_grads<OUT, ACC, false>;
      hipLaunchKernelGGL(grads, dim3(unsigned(dw_blocks + grid_dh)), dim3(kGemmNT), kGemmLdsBytes, s, dz, Wp, p.V_ld, dh_acc, dw_blocks,
                         dzT, hTc, V, H, total, p.tiles_v, tiles_h, p.T_pad, nact, vec_dw, dweight);
      const int64_t n = int64_t(V) * H;
      if (split.most > 1)
        hipLaunchKernelGGL((k_scatter_and_sum<OUT, ACC>), dim3(unsigned(T + (n / 8 + 255) / 256)), dim3(256), 0, s, dh_acc, pos, nact, H,
                           terms.scale, dh, unsigned(T), n, vec_dw, dweight);
      else
        hipLaunchKernelGGL(k_scatter_dh, dim3(unsigned(T)), dim3(256), 0, s, dh_acc, pos, nact, H, terms.scale, dh);
    };
    if (dw_bf16) accumulate ? launch(std::true_type{}, std::true_type{}) : launch(std::true_type{}, std::false_type{});
    else accumulate ? launch(std::false_type{}, std::true_type{}) : launch(std::false_type{}, std::false_type{});
    return launch_status();
  }
  if (T > 0) {
    hipLaunchKernelGGL(k_gemm_dh, dim3(unsigned(grid_dh)), dim3(kGemmNT), kGemmLdsBytes, s, dz, Wp, V, p.V_ld, H, tiles_h, nact, dh_acc);
    hipLaunchKernelGGL(k_scatter_dh, dim3(unsigned(T)), dim3(256), 0, s, dh_acc, pos, nact, H, terms.scale, dh);
  }
  // One launch where a workgroup walks (T == 0); where it has one tile, eight rounds of tiles a launch, so that the workgroups
  // that share operand slices stay close along K (32768 tokens at H = 3584, V = 152064, whole call: one launch 67.1, 16 rounds
  // 66.7, eight 66.1, four 66.8 ms; 16384 at H = 1536 even)
  const auto kernel = dw_bf16 ? (accumulate ? k_gemm_dw<true, true> : k_gemm_dw<true, false>)
                              : (accumulate ? k_gemm_dw<false, true> : k_gemm_dw<false, false>);
  const int per = p.T_pad < kDwTileRows ? total : 8 * cus;
  for (int t0 = 0; t0 < total; t0 += per) {
    const int n = total - t0 < per ? total - t0 : per;
    const dim3 grid = p.T_pad < kDwTileRows ? walkers(xcd_grid(n)) : dim3(unsigned(xcd_grid(n)));
    hipLaunchKernelGGL(kernel, grid, dim3(kGemmNT), kGemmLdsBytes, s, dzT, hTc, V, H, t0, n,
                       p.tiles_v, tiles_h, p.T_pad, nact, vec_dw, dweight);
  }
  return launch_status();
}
