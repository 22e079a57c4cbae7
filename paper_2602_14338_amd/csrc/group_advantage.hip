// Group statistics, curated subset, group-relative advantages and loss weights
// (Eq. 1; Sec. 3.2; Sec. 4.1 / Alg. 1 strata; Sec. 4.2 Strategies 2 and 3; App. C categories).
//
// Groups are ragged (CSR offsets).  One wave64 owns one group and walks it in strides of 64,
// so any group size works; counts are integers, the few floating-point statistics are formed
// in fp64 from those counts and rounded once to fp32.  The call is latency bound, so what counts is
// launches, dependent loads and exchanges between lanes:
//   up to 2048 groups and 8192 rollouts (a step)    k_curate: one launch, nothing passed between workgroups; without rejection
//                                                   up to 32768 rollouts of groups that fit a wave on average
//   up to 8192 groups                               k_group (c, category, keep mask, advantages, weights), then k_place:
//                                                   every workgroup adds up the kept counts in front of its groups
//                                                   itself, so no scan stands between
//   more                                            k_group, k_scan (exclusive scan of the kept counts, one
//                                                   workgroup) and k_compact: the counts would be read too often.
// Whole calls, k_group + k_place / k_curate, without rejection and with it: 256 groups of 16 6.6 / 4.2, 6.6 / 5.0 us; 256 of 32 6.6 / 4.2,
// 6.5 / 5.2; 64 of 128 6.6 / 6.0, 10.6 / 10.5; 16 of 500 12.8 / 12.6, 84 / 84.  Over 8192 rollouts, where a thread of 16 waves has 32 of the
// rewards in front to load, two launches are as fast where the host launches quickly and lose where it does not: 300 of 30 7.3 / 6.5, 7.7 / 7.5; 600 of 20
// 7.3 / 6.7, 7.5 / 7.3; 1000 of 32 7.4 / 6.6, 7.4 / 7.4; 2048 of 9 7.3 / 7.0, 7.5 / 7.7; 500 of 64 7.2 / 6.6, 7.4 / 7.8; on another box, without rejection,
// 6.6 / 6.7, 6.6 / 6.8, 6.6 / 6.8, 6.8 / 7.2.
// k_place / k_scan + k_compact: 400 groups (7831 rollouts) 9.0 / 11.4, 3000 (60325) 10.2 / 12.9, 4000 (80187) 11.0 / 14.5, 8000
// (159965) 18.1 / 24.1.  (Counting the bytes of the keep mask instead, up to 8192 rollouts, takes as long, and reads
// bytes that nobody wrote where offsets start above 0.)
// 100 groups of 64 to 90 rollouts, whose ranks do not fit one register a lane: 37.9 us when every lane looked for its
// rank by itself in memory, 10.4 with the candidates taken 64 at a time (ranks_before).
#include "aero_device.h"

namespace aero {

__device__ __forceinline__ float wave_max_f(float v) { return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); }); }
__device__ __forceinline__ float wave_min_f(float v) { return wave_reduce(v, [](float a, float b) { return fminf(a, b); }); }

constexpr int kGroupsPerBlock = 4;   // 4 waves of 64
constexpr int kPlaceQ = 1 << 13;     // k_place up to this many groups

// Category of a group of n rollouts of which c have reward exactly 1: u = c / n against tau, integer compares.
__device__ __forceinline__ int group_category(const aero_adv_params& p, int n, int c) {
  if (c == 0) return AERO_CAT_ZERO;
  if (c == n) return AERO_CAT_PERFECT;
  return int64_t(c) * p.tau_den < int64_t(n) * p.tau_num ? AERO_CAT_PARTIAL : AERO_CAT_GOOD;
}

// What is kept of it, known from n and c alone: everyone, nobody, every correct rollout and the m lowest-ranked incorrect ones,
// or the m lowest-ranked of the whole group.
enum KeepMode { kKeepAll, kKeepNone, kKeepCorrect, kKeepLowest };
struct KeepRule {
  KeepMode mode;
  int m, kept;
};
__device__ __forceinline__ KeepRule keep_rule(const aero_adv_params& p, int cat, int n, int c) {
  if (!p.reject_enable || cat == AERO_CAT_GOOD) return KeepRule{kKeepAll, 0, n};
  if (cat == AERO_CAT_PARTIAL) {
    const int m = int(min(int64_t(p.k_ratio) * c, int64_t(n - c)));
    return KeepRule{kKeepCorrect, m, c + m};
  }
  const int m = min(p.zero_keep, n);
  return p.posterior_mode ? KeepRule{kKeepLowest, m, m} : KeepRule{kKeepNone, 0, 0};
}

// Offsets outside [0, R] cannot make a kernel read out of bounds.
struct GroupRange {
  int b, e;
};
__device__ __forceinline__ GroupRange group_range(int lo, int hi, int R) {
  const int b = max(0, min(lo, R));
  return GroupRange{b, max(b, min(hi, R))};
}

// What a lane holds of its group's first 64 rollouts.
struct Held {
  float reward;
  uint32_t key;
  int length;
};
__device__ __forceinline__ Held load_held(GroupRange g, int lane, const float* __restrict__ rewards,
                                          const int32_t* __restrict__ lengths, const uint32_t* __restrict__ keys) {
  const int i = g.b + lane;
  if (i >= g.e) return Held{0.f, 0u, 0};
  return Held{rewards[i], keys ? keys[i] : 0u, lengths[i]};
}

// How many of the first n lanes' values (n <= 64, uniform) lie below `own`: every lane leaves its value in LDS and reads all of them, the
// same address in every lane.  (Handed round through the scalar side instead, a value at a time by v_readlane: a CU's waves share
// one scalar unit, and 16 groups of 32 rollouts were 4000 of its cycles.  Whole calls 256 groups of 8 to 32 6.7 / 4.7 us, with 8
// waves a workgroup; 8 of 32 5.0 / 3.5; 864 of 10 to 26, in two launches, 7.3 / 6.2.)
__device__ __forceinline__ int ranks_before(uint64_t* lds /*[64]*/, int lane, uint64_t value, int n, uint64_t own) {
  asm volatile("" ::: "memory");   // one wave's LDS accesses keep their order
  lds[lane] = value;
  asm volatile("" ::: "memory");
  int before = 0;
#pragma unroll 2
  for (int j = 0; j < n; j += 4) {   // uniform; values past n are ~0 or count for nobody
#pragma unroll
    for (int u = 0; u < 4; ++u) before += lds[j + u] < own;
  }
  return before;
}

// One group, one wave: everything but the position of its kept rollouts in kept_index.  Returns the
// number of kept rollouts (the same value in every lane); kept0: those among the group's first 64.
__device__ __forceinline__ int group_body(
    int q, GroupRange range, Held held, int lane, const float* __restrict__ rewards, const int32_t* __restrict__ lengths,
    const uint32_t* __restrict__ keys, int Q, const aero_adv_params& p, float* __restrict__ adv,
    float* __restrict__ weight, uint8_t* __restrict__ keep_mask, uint8_t* __restrict__ zero_var,
    uint8_t* __restrict__ category, int32_t* __restrict__ err_flag, uint64_t* ranks /*[64], LDS*/, uint64_t& kept0) {
  const int b = range.b, e = range.e;
  const int n = e - b;
  const bool curation = p.reject_enable || p.posterior_mode;

  // 1. c = number of rollouts with reward exactly 1
  const int i0 = b + lane;
  const bool in0 = i0 < e;
  const float r0 = held.reward;
  const uint32_t key0 = held.key;
  const int len0 = held.length;
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

  // 2. category, 3. kept subset
  const int cat = group_category(p, n, c);
  const KeepRule rule = keep_rule(p, cat, n, c);
  const KeepMode mode = rule.mode;
  const int m = rule.m;
  // a group that fits the wave: ranks from the lanes' own keys; smaller key first, ties to the lower index
  int ahead0 = 0;
  if (n <= kWave && mode >= kKeepCorrect) {
    const uint64_t in = __ballot(in0);
    uint64_t cand = in & (mode == kKeepLowest ? ~uint64_t(0) : ~ones);
    if (__popcll(cand) > m) {
      const uint64_t own = uint64_t(key0) << 32 | uint32_t(lane);
      ahead0 = ranks_before(ranks, lane, cand >> lane & 1 ? own : ~uint64_t(0), n, own);
    }
  }
  auto posterior_mean = [&]() { return (double(c) + double(p.alpha0)) / (double(n) + double(p.alpha0) + double(p.beta0)); };
  int nk;
  bool zv;
  if (n <= kWave && !bad) {
    // A group in the wave's registers whose rewards are 0 and 1 (every curated one): kept count, sum, extremes and
    // variance are counts of lanes.  With c correct and m incorrect rollouts kept, (1 - mean) / sigma = sqrt(m / c)
    // and -mean / sigma = -sqrt(c / m): no sums over the wave, one division and one root.
    const bool k = in0 && (mode == kKeepAll || (mode == kKeepCorrect && r0 == 1.f) || (mode >= kKeepCorrect && ahead0 < m));
    kept0 = __ballot(k);
    nk = __popcll(kept0);
    const int ck = __popcll(kept0 & ones);
    zv = ck == 0 || ck == nk;
    const bool one = r0 == 1.f;
    double a = 0.0;
    if (!zv) {
      const double up = double(one ? nk - ck : ck), down = double(one ? ck : nk - ck);
      a = sqrt(up / down);
      a = one ? a : -a;
    } else if (p.posterior_mode) {   // nk > 0 where a lane keeps anything
      const double mu = posterior_mean();
      a = (double(r0) - mu) * (1.0 / sqrt(mu * (1.0 - mu)));
    }
    if (in0) {
      keep_mask[i0] = k ? 1 : 0;
      adv[i0] = k ? float(a) : 0.f;
      weight[i0] = k && len0 > 0 ? float(1.0 / (double(Q) * double(nk) * double(len0))) : 0.f;
    }
  } else {
    bool keep0 = false;
    int nk_l = 0;                    // kept
    double sum_l = 0.0;              // sum of kept rewards
    float mx_l = -INFINITY, mn_l = INFINITY;
    auto take = [&](int i, float r, bool k) {
      keep_mask[i] = k ? 1 : 0;
      if (i == i0) keep0 = k;
      if (k) {
        ++nk_l;
        sum_l += double(r);
        mx_l = fmaxf(mx_l, r);
        mn_l = fminf(mn_l, r);
      }
    };
    if (mode < kKeepCorrect) {   // no ranks, and no exchange in the loop: loads of several steps go together
      for (int i = i0; i < e; i += kWave) take(i, i == i0 ? r0 : rewards[i], mode == kKeepAll);
    } else {
      for (int base = b; base < e; base += kWave) {   // uniform over the wave
        const int i = base + lane;
        const bool in = i < e;
        const float r = i == i0 ? r0 : in ? rewards[i] : 0.f;
        bool k = in && mode == kKeepCorrect && r == 1.f;
        if (n <= kWave) {
          k |= in && ahead0 < m;
        } else {
          // rank among the candidates (incorrect rollouts, or everyone), taken 64 at a time into the lanes
          const uint64_t own = uint64_t(in && keys ? keys[i] : 0u) << 32 | uint32_t(i);
          int ahead = 0;
          for (int from = b; from < e && __any(in && !k && ahead < m); from += kWave) {
            const int j0 = from + lane;
            const uint32_t kj = j0 < e && keys ? keys[j0] : 0u;
            const bool cand = j0 < e && (mode == kKeepLowest || rewards[j0] != 1.f);
            ahead += ranks_before(ranks, lane, cand ? uint64_t(kj) << 32 | uint32_t(j0) : ~uint64_t(0), kWave, own);
          }
          k |= in && ahead < m;
        }
        if (in) take(i, r, k);
      }
    }
    kept0 = __ballot(keep0);
    nk = wave_sum_i(nk_l);
    const float mx = wave_max_f(mx_l), mn = wave_min_f(mn_l);
    zv = nk == 0 || mx == mn;

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
      mu = posterior_mean();
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
  }
  if (lane == 0) {
    zero_var[q] = zv ? 1 : 0;
    category[q] = uint8_t(cat | (c <= p.s_rescue ? AERO_CAT_RESCUE_BIT : 0));
  }
  return nk;
}

// The kept ones among the 64 rollouts in the lanes (i: the lane's), ascending, from position `out` on.
__device__ __forceinline__ int place_kept(uint64_t kept, int i, int lane, int out, int R, int32_t* __restrict__ kept_index) {
  const int at = out + __popcll(kept & ((uint64_t(1) << lane) - 1));
  if ((kept >> lane & 1) && at < R) kept_index[at] = i;
  return __popcll(kept);
}

// Kept rollout indices of one group, ascending, written from position `out` on (one wave).  Groups that overlap can
// keep more than R rollouts between them: what does not fit kept_index is dropped.
__device__ __forceinline__ void compact_body(int q, int lane, const int32_t* __restrict__ group_offsets,
                                             const uint8_t* __restrict__ keep_mask, int out, int R,
                                             int32_t* __restrict__ kept_index) {
  const GroupRange g = group_range(group_offsets[q], group_offsets[q + 1], R);
  for (int base = g.b; base < g.e; base += kWave) {   // trip count is uniform over the wave
    const int i = base + lane;
    out += place_kept(__ballot(i < g.e && keep_mask[i] != 0), i, lane, out, R, kept_index);
  }
}

__global__ __launch_bounds__(kGroupsPerBlock* kWave) void k_group(
    const float* __restrict__ rewards, const int32_t* __restrict__ lengths,
    const int32_t* __restrict__ group_offsets, const uint32_t* __restrict__ keys, int Q, int R,
    aero_adv_params p, float* __restrict__ adv, float* __restrict__ weight, uint8_t* __restrict__ keep_mask,
    int32_t* __restrict__ kept_offsets, int count_mask, uint8_t* __restrict__ zero_var, uint8_t* __restrict__ category,
    int32_t* __restrict__ err_flag) {
  __shared__ __align__(16) uint64_t ranks[kGroupsPerBlock][kWave];
  const int lane = threadIdx.x % kWave;
  const int q = blockIdx.x * kGroupsPerBlock + threadIdx.x / kWave;
  if (q >= Q) return;   // whole wave leaves together
  const GroupRange range = group_range(group_offsets[q], group_offsets[q + 1], R);
  uint64_t kept0;
  const int nk = group_body(q, range, load_held(range, lane, rewards, lengths, keys), lane, rewards, lengths, keys, Q, p, adv,
                            weight, keep_mask, zero_var, category, err_flag, ranks[threadIdx.x / kWave], kept0);
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

// All of it in one launch: a wave per group, up to WAVES in a workgroup.  Eight (16 or 4: 5.1 us for 256 groups of 8 to 32 where 8
// take 4.7) but for more than kCurateManyQ groups, where half as many workgroups read the rewards in front and each goes over
// the groups in front in half the turns: 8 / 16 waves, with rejection and without, 2048 groups of 2 5.39 / 5.28, 5.19 / 5.06 us; 1700 of 3 5.72 /
// 5.55, 5.35 / 5.20; 1500 of 5 5.55 / 5.64, 5.18 / 5.19; 850 of 8 5.10 / 5.22, 4.74 / 4.72; 512 of 8 4.43 / 4.80, 4.11 / 4.30.  How many rollouts a group keeps follows from its size
// and its count of correct rollouts alone, so a workgroup counts what lies in front of its groups itself, from the
// rewards (a bit per rollout in LDS, a thread per group), while its own groups' loads are under way; nothing is passed
// between workgroups.  Bound by latency: kernel arguments, offsets, rewards, and the instructions themselves, which come
// from memory once per launch.
constexpr int kCurateR = 8192, kCurateWideR = 32768, kCurateQ = 2048, kCurateManyQ = 1536;
// LOADS: rewards per thread, all in flight at once; R <= LOADS * WAVES * 64 unless there is one workgroup.
template <int WAVES, int LOADS>
__global__ __launch_bounds__(WAVES* kWave) void k_curate(
    const float* __restrict__ rewards, const int32_t* __restrict__ lengths,
    const int32_t* __restrict__ group_offsets, const uint32_t* __restrict__ keys, int Q, int R,
    aero_adv_params p, float* __restrict__ adv, float* __restrict__ weight, uint8_t* __restrict__ keep_mask,
    int32_t* __restrict__ kept_index, int32_t* __restrict__ kept_offsets, uint8_t* __restrict__ zero_var,
    uint8_t* __restrict__ category, int32_t* __restrict__ err_flag) {
  constexpr int NT = WAVES * kWave;
  __shared__ uint64_t ones[LOADS * WAVES];   // bit i % 64 of word i / 64: reward i is exactly 1
  __shared__ int front[WAVES], own[WAVES];
  __shared__ __align__(16) uint64_t ranks[WAVES][kWave];
  const int tid = threadIdx.x, lane = tid % kWave, wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int waves = blockDim.x / kWave;
  const int q0 = blockIdx.x * waves, q = q0 + wave;
  // Loads that depend on nothing come first, from clamped positions so that no branch stands between them; what lies
  // past the end is not looked at.
  int ahead_b = 0, ahead_e = 0;
  float x[LOADS];
  if (q0 > 0 && R > 0) {   // uniform; then there are NT threads
#pragma unroll
    for (int u = 0; u < LOADS; ++u) x[u] = rewards[min(u * NT + tid, R - 1)];
    const int at = min(tid, q0 - 1);
    ahead_b = group_offsets[at];
    ahead_e = group_offsets[at + 1];
  }
  const int qc = min(q, Q - 1);
  GroupRange mine = group_range(group_offsets[qc], group_offsets[qc + 1], R);
  if (q >= Q) mine.e = mine.b;
  const Held held = load_held(mine, lane, rewards, lengths, keys);
  int before_me = 0;
  if (q0 > 0 && R > 0) {
#pragma unroll
    for (int u = 0; u < LOADS; ++u) {
      const uint64_t bits = __ballot(x[u] == 1.f);
      if (lane == 0) ones[u * WAVES + wave] = bits;
    }
    __syncthreads();
#pragma unroll 1
    for (int at = tid; at - tid < q0; at += NT) {   // uniform
      GroupRange g = group_range(ahead_b, ahead_e, R);
      if (at >= q0) g.e = g.b;
      if (at - tid + NT < q0) {   // the next one's
        const int next = min(at + NT, q0 - 1);
        ahead_b = group_offsets[next];
        ahead_e = group_offsets[next + 1];
      }
      int c = 0;
      for (int w = g.b / 64; w * 64 < g.e; ++w) {
        uint64_t bits = ones[w];
        if (w * 64 < g.b) bits &= ~uint64_t(0) << (g.b % 64);
        if (g.e - w * 64 < 64) bits &= ~(~uint64_t(0) << (g.e % 64));
        c += __popcll(bits);
      }
      const int n = g.e - g.b;
      before_me += keep_rule(p, group_category(p, n, c), n, c).kept;   // an empty group keeps none
    }
    before_me = wave_sum_i(before_me);
  }
  uint64_t kept0 = 0;
  int nk = 0;
  if (q < Q)   // uniform over the wave
    nk = group_body(q, mine, held, lane, rewards, lengths, keys, Q, p, adv, weight, keep_mask, zero_var, category, err_flag, ranks[wave], kept0);
  if (lane == 0) {
    front[wave] = before_me;
    own[wave] = nk;
  }
  __syncthreads();
  int out = wave_sum_i(lane < waves ? front[lane] + (lane < wave ? own[lane] : 0) : 0);
  if (q >= Q) return;
  if (lane == 0) {
    if (q == 0) kept_offsets[0] = 0;
    kept_offsets[q + 1] = out + nk;
  }
  out += place_kept(kept0, mine.b + lane, lane, out, R, kept_index);
  for (int base = mine.b + kWave; base < mine.e; base += kWave) {   // a long group: the mask its own lanes wrote
    const int i = base + lane;
    out += place_kept(__ballot(i < mine.e && keep_mask[i] != 0), i, lane, out, R, kept_index);
  }
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
  const bool few = R <= kCurateR, ranks = p->reject_enable;
  if (Q > 0 && Q <= kCurateQ && (few || (R <= kCurateWideR && R <= kWave * Q && !ranks))) {   // see the top
    const int most = few && Q <= kCurateManyQ ? 8 : 16, waves = Q < most ? Q : most;
    const auto kernel = !few        ? k_curate<16, kCurateWideR / (16 * kWave)>
                        : most == 8 ? k_curate<8, kCurateR / (8 * kWave)>
                                    : k_curate<16, kCurateR / (16 * kWave)>;
    hipLaunchKernelGGL(kernel, dim3(unsigned((Q + waves - 1) / waves)), dim3(unsigned(waves * kWave)), 0, s, rewards, lengths,
                       group_offsets, keep_priority, Q, R, *p, adv, weight, keep_mask, kept_index, kept_offsets, group_zero_var,
                       group_category, err_flag);
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
