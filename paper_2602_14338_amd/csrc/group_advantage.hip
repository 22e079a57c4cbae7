// Group statistics, curated subset, group-relative advantages and loss weights
// (Eq. 1; Sec. 3.2; Sec. 4.1 / Alg. 1 strata; Sec. 4.2 Strategies 2 and 3; App. C categories).
//
// Groups are ragged (CSR offsets).  One wave64 owns one group and walks it in strides of 64,
// so any group size works; counts are integers, the few floating-point statistics are formed
// in fp64 from those counts and rounded once to fp32.  The call is latency bound, so what counts is
// launches and dependent loads:
//   at most 32 groups (a micro-batch)   k_group_small: everything in one workgroup, one launch
//   up to 8192 groups (a step)          k_group (c, category, keep mask, advantages, weights), then k_place:
//                                       every workgroup adds up the kept counts in front of its groups
//                                       itself, so no scan stands between
//   more                                k_group, k_scan (exclusive scan of the kept counts, one
//                                       workgroup) and k_compact: the counts would be read too often.
// Whole calls, k_place against the last two kernels: 64 groups (1024 rollouts) 8.8 / 11.2 us, 400 (7831) 9.0 / 11.4,
// 410 (8296) 8.9 / 11.3, 600 (12108) 9.0 / 11.3, 1500 (24384) 9.3 / 11.6, 3000 (60325) 10.2 / 12.9, 4000 (80187)
// 11.0 / 14.5, 8000 (159965) 18.1 / 24.1.  (Counting the bytes of the keep mask instead, up to 8192 rollouts,
// takes as long, and reads bytes that nobody wrote where offsets start above 0.)
// 256 groups of 8 to 32 rollouts took 15.8 us with the third form and a rank search that loaded rewards and
// keys one at a time; a group of at most 64 rollouts now stays in the lanes of its wave.  (One workgroup
// for 64 groups serialises them: 18.7 us against 13.5.)
#include "aero_device.h"

namespace aero {

__device__ __forceinline__ int wave_sum_i(int v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}
__device__ __forceinline__ int wave_max_i(int v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, kWave));
  return v;
}
__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
  return v;
}
__device__ __forceinline__ float wave_max_f(float v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
  return v;
}
__device__ __forceinline__ float wave_min_f(float v) {
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off, kWave));
  return v;
}

// (key, index) ordering used for down-sampling: smaller key first, ties to the lower index
__device__ __forceinline__ bool before(uint32_t ka, int ia, uint32_t kb, int ib) {
  return ka < kb || (ka == kb && ia < ib);
}

constexpr int kGroupsPerBlock = 4;   // 4 waves of 64
constexpr int kPlaceQ = 1 << 13;     // k_place up to this many groups (see the top)

// One group, one wave: everything but the position of its kept rollouts in kept_index.  Returns the
// number of kept rollouts (the same value in every lane).
__device__ __forceinline__ int group_body(
    int q, int lane, const float* __restrict__ rewards, const int32_t* __restrict__ lengths,
    const int32_t* __restrict__ group_offsets, const uint32_t* __restrict__ keys, int Q, int R,
    const aero_adv_params& p, float* __restrict__ adv, float* __restrict__ weight, uint8_t* __restrict__ keep_mask,
    uint8_t* __restrict__ zero_var, uint8_t* __restrict__ category, int32_t* __restrict__ err_flag) {
  int b = group_offsets[q], e = group_offsets[q + 1];
  b = max(0, min(b, R));   // offsets outside [0, R] cannot make the kernel read out of bounds
  e = max(b, min(e, R));
  const int n = e - b;
  const bool curation = p.reject_enable || p.posterior_mode;

  // 1. c = number of rollouts with reward exactly 1; what the lane's first rollout holds, loaded at once
  const int i0 = b + lane;
  const bool in0 = i0 < e;
  const float r0 = in0 ? rewards[i0] : 0.f;
  const uint32_t key0 = in0 && keys ? keys[i0] : 0u;
  const int len0 = in0 ? lengths[i0] : 0;
  const uint64_t ones = __ballot(in0 && r0 == 1.f);   // of the group's first 64 rollouts
  int c = __popcll(ones);
  bool bad = __ballot(in0 && r0 != 0.f && r0 != 1.f) != 0;
  if (n > kWave) {
    int c_l = 0, bad_l = 0;
    for (int i = i0 + kWave; i < e; i += kWave) {
      const float r = rewards[i];
      c_l += r == 1.f;
      bad_l += (r != 0.f && r != 1.f);
    }
    c += wave_sum_i(c_l);
    bad |= wave_sum_i(bad_l) != 0;
  }
  if (curation && bad && lane == 0 && err_flag) atomicOr(err_flag, AERO_DERR_NONBINARY_REWARD);

  // 2. category by u = c/n against tau, integer compares
  int cat;
  if (c == 0) cat = AERO_CAT_ZERO;
  else if (c == n) cat = AERO_CAT_PERFECT;
  else if (int64_t(c) * p.tau_den < int64_t(n) * p.tau_num) cat = AERO_CAT_PARTIAL;
  else cat = AERO_CAT_GOOD;

  // 3. kept subset.  mode 0: all, 1: none, 2: all correct + m lowest-ranked incorrect,
  //    3: the m lowest-ranked of the whole group
  int mode = 0, m = 0;
  if (p.reject_enable) {
    if (cat == AERO_CAT_PARTIAL) {
      mode = 2;
      m = int(min(int64_t(p.k_ratio) * c, int64_t(n - c)));
    } else if (cat != AERO_CAT_GOOD) {
      mode = p.posterior_mode ? 3 : 1;
      m = min(p.zero_keep, n);
    }
  }
  bool keep0 = false;
  int nk_l = 0;                    // kept
  double sum_l = 0.0;              // sum of kept rewards
  // a group that fits the wave: ranks from the lanes' registers, one candidate of the group at a time
  int ahead0 = 0;
  if (n <= kWave && mode >= 2) {
    uint64_t cand = __ballot(in0) & (mode == 3 ? ~uint64_t(0) : ~ones);
    while (cand) {   // uniform
      const int j = __ffsll((unsigned long long)cand) - 1;
      cand &= cand - 1;
      ahead0 += before(uint32_t(__builtin_amdgcn_readlane(int(key0), j)), j, key0, lane);
    }
  }
  float mx_l = -INFINITY, mn_l = INFINITY;
  for (int i = b + lane; i < e; i += kWave) {
    const float r = i == i0 ? r0 : rewards[i];
    bool k;
    if (mode == 0) k = true;
    else if (mode == 1) k = false;
    else if (mode == 2 && r == 1.f) k = true;
    else if (n <= kWave) k = ahead0 < m;
    else {
      // rank among the candidates (incorrect rollouts in mode 2, everyone in mode 3)
      const uint32_t ki = keys ? keys[i] : 0u;
      int ahead = 0;
      for (int j = b; j < e && ahead < m; ++j) {
        const bool cand = mode == 3 || rewards[j] != 1.f;
        ahead += cand && before(keys ? keys[j] : 0u, j, ki, i);
      }
      k = ahead < m;
    }
    keep_mask[i] = k ? 1 : 0;
    if (i == i0) keep0 = k;
    if (k) {
      ++nk_l;
      sum_l += double(r);
      mx_l = fmaxf(mx_l, r);
      mn_l = fminf(mn_l, r);
    }
  }
  const int nk = wave_sum_i(nk_l);
  const float mx = wave_max_f(mx_l), mn = wave_min_f(mn_l);
  const bool zv = nk == 0 || mx == mn;

  // 4./5. advantages over the kept subset
  double mu = 0.0, inv_sigma = 0.0;
  if (!zv) {
    mu = wave_sum_d(sum_l) / double(nk);
    double ss_l = 0.0;
    for (int i = b + lane; i < e; i += kWave)
      if (i == i0 ? keep0 : keep_mask[i] != 0) {   // written by this same lane above
        const double d = double(i == i0 ? r0 : rewards[i]) - mu;
        ss_l += d * d;
      }
    inv_sigma = 1.0 / sqrt(wave_sum_d(ss_l) / double(nk));
  } else if (p.posterior_mode && nk > 0) {
    // posterior mean from the observed c, n of the whole group
    mu = (double(c) + double(p.alpha0)) / (double(n) + double(p.alpha0) + double(p.beta0));
    inv_sigma = 1.0 / sqrt(mu * (1.0 - mu));
  }
  const bool signal = !zv || (p.posterior_mode && nk > 0);

  // 6. weights 1 / (Q n' L_i)
  for (int i = b + lane; i < e; i += kWave) {
    const bool k = i == i0 ? keep0 : keep_mask[i] != 0;
    float a = 0.f, w = 0.f;
    if (k) {
      if (signal) a = float((double(i == i0 ? r0 : rewards[i]) - mu) * inv_sigma);
      const int L = i == i0 ? len0 : lengths[i];
      if (L > 0) w = float(1.0 / (double(Q) * double(nk) * double(L)));
    }
    adv[i] = a;
    weight[i] = w;
  }
  if (lane == 0) {
    zero_var[q] = zv ? 1 : 0;
    category[q] = uint8_t(cat | (c <= p.s_rescue ? AERO_CAT_RESCUE_BIT : 0));
  }
  return nk;
}

// Kept rollout indices of one group, ascending, written from position `out` on (one wave).  Groups that overlap can
// keep more than R rollouts between them: what does not fit kept_index is dropped.
__device__ __forceinline__ void compact_body(int q, int lane, const int32_t* __restrict__ group_offsets,
                                             const uint8_t* __restrict__ keep_mask, int out, int R,
                                             int32_t* __restrict__ kept_index) {
  int b = group_offsets[q], e = group_offsets[q + 1];
  b = max(0, min(b, R));
  e = max(b, min(e, R));
  for (int base = b; base < e; base += kWave) {   // trip count is uniform over the wave
    const int i = base + lane;
    const bool k = i < e && keep_mask[i] != 0;
    const uint64_t bal = __ballot(k);
    const int at = out + __popcll(bal & ((uint64_t(1) << lane) - 1));
    if (k && at < R) kept_index[at] = i;
    out += __popcll(bal);
  }
}

__global__ __launch_bounds__(kGroupsPerBlock* kWave) void k_group(
    const float* __restrict__ rewards, const int32_t* __restrict__ lengths,
    const int32_t* __restrict__ group_offsets, const uint32_t* __restrict__ keys, int Q, int R,
    aero_adv_params p, float* __restrict__ adv, float* __restrict__ weight, uint8_t* __restrict__ keep_mask,
    int32_t* __restrict__ kept_offsets, int count_mask, uint8_t* __restrict__ zero_var, uint8_t* __restrict__ category,
    int32_t* __restrict__ err_flag) {
  const int lane = threadIdx.x % kWave;
  const int q = blockIdx.x * kGroupsPerBlock + threadIdx.x / kWave;
  if (q >= Q) return;   // whole wave leaves together
  const int nk = group_body(q, lane, rewards, lengths, group_offsets, keys, Q, R, p, adv, weight, keep_mask, zero_var,
                            category, err_flag);
  if (lane == 0) kept_offsets[q + 1] = nk ^ count_mask;   // count_mask: 0, or -1 for k_place
}

// Exclusive scan of counts held in kept_offsets[1..Q] (in place), kept_offsets[0] = 0.
constexpr int kScanNT = 1024;
__global__ __launch_bounds__(kScanNT) void k_scan(int32_t* kept_offsets, int Q) {
  __shared__ int part[kScanNT];
  const int per = (Q + kScanNT - 1) / kScanNT;
  const int lo = min(Q, int(threadIdx.x) * per), hi = min(Q, lo + per);
  int s = 0;
  for (int q = lo; q < hi; ++q) s += kept_offsets[q + 1];
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = 1; off < kScanNT; off <<= 1) {   // inclusive Hillis-Steele over thread sums
    int v = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
    __syncthreads();
    part[threadIdx.x] += v;
    __syncthreads();
  }
  int run = threadIdx.x ? part[threadIdx.x - 1] : 0;
  for (int q = lo; q < hi; ++q) {
    run += kept_offsets[q + 1];
    kept_offsets[q + 1] = run;
  }
  if (threadIdx.x == 0) kept_offsets[0] = 0;
}

__global__ __launch_bounds__(kGroupsPerBlock* kWave) void k_compact(
    const int32_t* __restrict__ group_offsets, const uint8_t* __restrict__ keep_mask,
    const int32_t* __restrict__ kept_offsets, int Q, int R, int32_t* __restrict__ kept_index) {
  const int lane = threadIdx.x % kWave;
  const int q = blockIdx.x * kGroupsPerBlock + threadIdx.x / kWave;
  if (q >= Q) return;
  compact_body(q, lane, group_offsets, keep_mask, kept_offsets[q], R, kept_index);
}

// kept_offsets and kept_index from the counts that k_group left in kept_offsets, without a scan in between: a
// workgroup adds up the counts in front of its four groups by itself.  Workgroups that are through replace counts by
// offsets meanwhile, so counts are stored as ~count: a negative entry is a count, any other the offset behind that
// group, and an offset stands for everything in front of it.  Whatever mixture a workgroup sees, the last offset
// plus the counts behind it is the sum it is after.
constexpr int kPlaceNT = kGroupsPerBlock * kWave;
// LOADS: counts per thread, all in flight at once; Q <= LOADS * kPlaceNT.
template <int LOADS>
__global__ __launch_bounds__(kPlaceNT) void k_place(
    const int32_t* __restrict__ group_offsets, const uint8_t* __restrict__ keep_mask, int Q, int R,
    int32_t* kept_offsets, int32_t* __restrict__ kept_index) {
  __shared__ int last[kGroupsPerBlock], front[kGroupsPerBlock], own[kGroupsPerBlock];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int q0 = blockIdx.x * kGroupsPerBlock, q = q0 + wave;
  auto entry = [&](int p) { return __hip_atomic_load(kept_offsets + p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
  int v[LOADS];
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    const int p = u * kPlaceNT + tid;
    v[u] = -1;   // a count of 0
    if (u * kPlaceNT < q0 && p < q0) v[u] = entry(p);
  }
  const int mine = q < Q ? ~entry(q) : 0;   // nobody else replaces it
  int n = 0;
  bool offset_seen = false;
#pragma unroll
  for (int u = 0; u < LOADS; ++u) {
    n += ~v[u];
    offset_seen |= v[u] >= 0;
  }
  n = wave_sum_i(n);
  const int seen = __any(offset_seen);
  if (lane == 0) {
    front[wave] = n;
    last[wave] = seen;
    own[wave] = mine;
  }
  __syncthreads();
  static_assert(kGroupsPerBlock == 4, "four flags");
  if (last[0] | last[1] | last[2] | last[3]) {   // uniform: counts from the last offset on
    int at = -1;
#pragma unroll
    for (int u = 0; u < LOADS; ++u)
      if (v[u] >= 0) at = u * kPlaceNT + tid;
    at = wave_max_i(at);
    __syncthreads();   // the flags have been read
    if (lane == 0) last[wave] = at;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kGroupsPerBlock; ++w) at = max(at, last[w]);
    n = 0;
#pragma unroll
    for (int u = 0; u < LOADS; ++u)
      if (u * kPlaceNT + tid >= at) n += v[u] < 0 ? ~v[u] : v[u];   // at itself: the offset
    n = wave_sum_i(n);
    if (lane == 0) front[wave] = n;
    __syncthreads();
  }
  int out = 0;
#pragma unroll
  for (int w = 0; w < kGroupsPerBlock; ++w) out += front[w] + (w < wave ? own[w] : 0);
  if (q >= Q) return;
  if (lane == 0) {
    if (q == 0) kept_offsets[0] = 0;
    __hip_atomic_store(kept_offsets + q + 1, out + mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  compact_body(q, lane, group_offsets, keep_mask, out, R, kept_index);
}

// The three stages in one workgroup of 16 waves, for Q <= kSmallQ groups: wave w takes groups w and w + 16;
// the kept counts and their scan stay in LDS; every wave then places the kept indices of the groups it
// processed (it reads back the keep mask its own lanes wrote).
constexpr int kSmallQ = 32, kSmallR = 1 << 16, kSmallNT = 1024;
__global__ __launch_bounds__(kSmallNT) void k_group_small(
    const float* __restrict__ rewards, const int32_t* __restrict__ lengths,
    const int32_t* __restrict__ group_offsets, const uint32_t* __restrict__ keys, int Q, int R,
    aero_adv_params p, float* __restrict__ adv, float* __restrict__ weight, uint8_t* __restrict__ keep_mask,
    int32_t* __restrict__ kept_index, int32_t* __restrict__ kept_offsets, uint8_t* __restrict__ zero_var,
    uint8_t* __restrict__ category, int32_t* __restrict__ err_flag) {
  __shared__ int start[kSmallQ + 1];   // counts, then exclusive offsets
  __shared__ int part[kSmallNT / kWave];
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  constexpr int kWaves = kSmallNT / kWave;
  for (int q = wave; q < Q; q += kWaves) {
    const int nk = group_body(q, lane, rewards, lengths, group_offsets, keys, Q, R, p, adv, weight, keep_mask, zero_var,
                              category, err_flag);
    if (lane == 0) start[q] = nk;
  }
  __syncthreads();
  // exclusive scan of start[0 .. Q): two entries per thread, shuffles inside a wave, the 16 wave totals through LDS
  const int q0 = 2 * tid, q1 = 2 * tid + 1;
  const int c0 = q0 < Q ? start[q0] : 0, c1 = q1 < Q ? start[q1] : 0;
  int incl = c0 + c1;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const int v = __shfl_up(incl, off, kWave);
    if (lane >= off) incl += v;
  }
  if (lane == kWave - 1) part[wave] = incl;
  __syncthreads();   // also: every read of start[] above precedes the writes below
  int before_me = incl - (c0 + c1), total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    before_me += w < wave ? part[w] : 0;
    total += part[w];
  }
  if (q0 < Q) start[q0] = before_me;
  if (q1 < Q) start[q1] = before_me + c0;
  if (tid == 0) start[Q] = total;
  __syncthreads();
  for (int q = tid; q <= Q; q += kSmallNT) kept_offsets[q] = start[q];
  for (int q = wave; q < Q; q += kWaves) compact_body(q, lane, group_offsets, keep_mask, start[q], R, kept_index);
}

}  // namespace aero

extern "C" aero_status aero_group_advantage(
    const float* rewards, const int32_t* lengths, const int32_t* group_offsets,
    const uint32_t* keep_priority, int32_t Q, int32_t R, const aero_adv_params* p, float* adv,
    float* weight, uint8_t* keep_mask, int32_t* kept_index, int32_t* kept_offsets,
    uint8_t* group_zero_var, uint8_t* group_category, int32_t* err_flag, void* stream) {
  using namespace aero;
  if (Q < 0 || R < 0) return AERO_ERR_SHAPE;
  if (!p || !group_offsets || !kept_offsets) return AERO_ERR_NULL;
  if (p->k_ratio < 1 || p->tau_den < 1 || p->tau_num < 0 || p->zero_keep < 0 || p->s_rescue < 0) return AERO_ERR_SHAPE;
  if (Q > 0 && (!group_zero_var || !group_category)) return AERO_ERR_NULL;
  if (R > 0 && (!rewards || !lengths || !adv || !weight || !keep_mask || !kept_index)) return AERO_ERR_NULL;
  hipStream_t s = as_stream(stream);
  if (Q > 0 && Q <= kSmallQ && R <= kSmallR) {
    hipLaunchKernelGGL(k_group_small, dim3(1), dim3(kSmallNT), 0, s, rewards, lengths, group_offsets, keep_priority, Q, R,
                       *p, adv, weight, keep_mask, kept_index, kept_offsets, group_zero_var, group_category, err_flag);
    return launch_status();
  }
  const unsigned blocks = unsigned((Q + kGroupsPerBlock - 1) / kGroupsPerBlock);
  const bool place = Q > 0 && Q <= kPlaceQ;
  if (Q > 0)
    hipLaunchKernelGGL(k_group, dim3(blocks), dim3(kGroupsPerBlock * kWave), 0, s, rewards, lengths, group_offsets,
                       keep_priority, Q, R, *p, adv, weight, keep_mask, kept_offsets, place ? -1 : 0, group_zero_var,
                       group_category, err_flag);
  if (place) {
    // sixteen loads do for 4096 groups; thirty-two everywhere cost 0.5 us
    const auto kernel = Q <= 16 * kPlaceNT ? k_place<16> : k_place<kPlaceQ / kPlaceNT>;
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kGroupsPerBlock * kWave), 0, s, group_offsets, keep_mask, Q, R,
                       kept_offsets, kept_index);
    return launch_status();
  }
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanNT), 0, s, kept_offsets, Q);
  if (Q > 0)
    hipLaunchKernelGGL(k_compact, dim3(blocks), dim3(kGroupsPerBlock * kWave), 0, s, group_offsets, keep_mask,
                       kept_offsets, Q, R, kept_index);
  return launch_status();
}
