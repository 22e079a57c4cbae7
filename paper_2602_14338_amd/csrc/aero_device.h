// Device-side helpers shared by the kernels: bf16 packing, wave64 reductions,
// the running (max, sum-exp, sum-exp-times-logit) state of a softmax row.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "../../include/aero.h"

namespace aero {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kWave = 64;

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));   // one 16-byte global access

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ float bf16_to_f32(uint16_t b) { return __uint_as_float(uint32_t(b) << 16); }

// two floats -> packed bf16 pair, round-to-nearest-even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2_t f = {lo, hi};
  bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
  return *reinterpret_cast<uint32_t*>(&b);
}
__device__ __forceinline__ uint16_t f32_to_bf16(float x) {
  return uint16_t(pack_bf16x2(x, 0.f) & 0xffffu);
}

// IEEE binary16 storage: widening is exact, narrowing rounds to nearest even (subnormals kept).
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float f16_to_f32(uint16_t b) {
  _Float16 h;
  __builtin_memcpy(&h, &b, 2);
  return float(h);
}
__device__ __forceinline__ uint32_t pack_f16x2(float lo, float hi) {
  f32x2_t f = {lo, hi};
  f16x2_t h = __builtin_convertvector(f, f16x2_t);
  uint32_t w;
  __builtin_memcpy(&w, &h, 4);
  return w;
}
__device__ __forceinline__ uint16_t f32_to_f16(float x) { return uint16_t(pack_f16x2(x, 0.f) & 0xffffu); }

// 8-bit float storage, 4 exponent and 3 mantissa bits, no infinities (largest finite value 448): widening is
// exact; narrowing rounds to nearest even, keeps subnormals (multiples of 2^-9) and saturates beyond +-448.
__device__ __forceinline__ float f8_to_f32(uint8_t b) { return __builtin_amdgcn_cvt_f32_fp8(int(b), 0); }
__device__ __forceinline__ uint32_t pack_f8x4(float a, float b, float c, float d) {
  constexpr float kMax = 448.f;
  a = __builtin_amdgcn_fmed3f(a, -kMax, kMax);
  b = __builtin_amdgcn_fmed3f(b, -kMax, kMax);
  c = __builtin_amdgcn_fmed3f(c, -kMax, kMax);
  d = __builtin_amdgcn_fmed3f(d, -kMax, kMax);
  int p = 0;
  p = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, p, false);   // low half of the word
  p = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, p, true);    // high half
  return uint32_t(p);
}
__device__ __forceinline__ uint8_t f32_to_f8(float x) { return uint8_t(pack_f8x4(x, 0.f, 0.f, 0.f) & 0xffu); }

// Storage type tags (the values of the public dtype codes) and what depends on them.
constexpr int kF32 = AERO_F32, kBF16 = AERO_BF16, kF16 = AERO_F16, kF8 = AERO_F8E4M3;
template <int DT> struct Storage {
  static constexpr int kBytes = DT == kF32 ? 4 : DT == kF8 ? 1 : 2;
  static constexpr int kPerVec = 16 / kBytes;   // elements per 16-byte vector
  static constexpr int kLogPerVec = DT == kF32 ? 2 : DT == kF8 ? 4 : 3;
};
inline bool storage_dtype_ok(int32_t dtype) {
  return dtype == AERO_BF16 || dtype == AERO_F32 || dtype == AERO_F16 || dtype == AERO_F8E4M3;
}
inline size_t storage_bytes(int32_t dtype) { return dtype == AERO_F32 ? 4 : dtype == AERO_F8E4M3 ? 1 : 2; }
template <int DT> __device__ __forceinline__ float load_elt(const void* row, int64_t j) {
  if constexpr (DT == kBF16) return bf16_to_f32(reinterpret_cast<const uint16_t*>(row)[j]);
  else if constexpr (DT == kF16) return f16_to_f32(reinterpret_cast<const uint16_t*>(row)[j]);
  else if constexpr (DT == kF8) return f8_to_f32(reinterpret_cast<const uint8_t*>(row)[j]);
  else return reinterpret_cast<const float*>(row)[j];
}
template <int DT> __device__ __forceinline__ void store_elt(void* row, int64_t j, float x) {
  if constexpr (DT == kBF16) reinterpret_cast<uint16_t*>(row)[j] = f32_to_bf16(x);
  else if constexpr (DT == kF16) reinterpret_cast<uint16_t*>(row)[j] = f32_to_f16(x);
  else if constexpr (DT == kF8) reinterpret_cast<uint8_t*>(row)[j] = f32_to_f8(x);
  else reinterpret_cast<float*>(row)[j] = x;
}

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// Softmax row state relative to an offset m (any m close enough to the row maximum that
// nothing overflows): s = sum exp(z - m), sz = sum exp(z - m) z.
struct RowStat {
  float m, s, sz;
};

__device__ __forceinline__ RowStat stat_identity() { return RowStat{-INFINITY, 0.f, 0.f}; }

__device__ __forceinline__ RowStat stat_merge(RowStat a, RowStat b) {
  float M = fmaxf(a.m, b.m);
  float fa = (a.m == M) ? 1.f : exp2_fast((a.m - M) * kLog2e);
  float fb = (b.m == M) ? 1.f : exp2_fast((b.m - M) * kLog2e);
  return RowStat{M, a.s * fa + b.s * fb, a.sz * fa + b.sz * fb};
}

__device__ __forceinline__ RowStat stat_shfl_xor(RowStat a, int mask) {
  return RowStat{__shfl_xor(a.m, mask, kWave), __shfl_xor(a.s, mask, kWave), __shfl_xor(a.sz, mask, kWave)};
}

// All-reduce over the 16 lanes of a row, or over the wave, by lane permutations of the vector ALU (no LDS
// round trips).  The mirrors stand for exchanges at distance 4 and 8: the lanes they mix are equal by then.
template <int CTRL> __device__ __forceinline__ float dpp_move(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xf, 0xf, true));
}
template <class Op> __device__ __forceinline__ float row16_reduce(float x, Op op) {
  x = op(x, dpp_move<0xB1>(x));    // quad_perm [1,0,3,2]
  x = op(x, dpp_move<0x4E>(x));    // quad_perm [2,3,0,1]
  x = op(x, dpp_move<0x141>(x));   // row_half_mirror
  return op(x, dpp_move<0x140>(x));   // row_mirror
}
template <class Op> __device__ __forceinline__ float wave_reduce(float x, Op op) {
  x = row16_reduce(x, op);
  const auto r16 = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = op(__uint_as_float(r16[0]), __uint_as_float(r16[1]));
  const auto r32 = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return op(__uint_as_float(r32[0]), __uint_as_float(r32[1]));
}

// The same exchanges for integers and for 64-bit floats (in two halves): a fixed order, the same result in every lane.
template <int CTRL> __device__ __forceinline__ int dpp_move_i(int x) { return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xf, 0xf, true); }
template <class Op> __device__ __forceinline__ int wave_reduce_i(int v, Op op) {
  v = op(v, dpp_move_i<0xB1>(v));
  v = op(v, dpp_move_i<0x4E>(v));
  v = op(v, dpp_move_i<0x141>(v));
  v = op(v, dpp_move_i<0x140>(v));
  const auto r16 = __builtin_amdgcn_permlane16_swap(uint32_t(v), uint32_t(v), false, false);
  v = op(int(r16[0]), int(r16[1]));
  const auto r32 = __builtin_amdgcn_permlane32_swap(uint32_t(v), uint32_t(v), false, false);
  return op(int(r32[0]), int(r32[1]));
}
__device__ __forceinline__ int wave_sum_i(int v) { return wave_reduce_i(v, [](int a, int b) { return a + b; }); }
__device__ __forceinline__ int wave_max_i(int v) { return wave_reduce_i(v, [](int a, int b) { return max(a, b); }); }
__device__ __forceinline__ double wave_sum_d(double v) {
  auto both = [](int lo, int hi) { return __hiloint2double(hi, lo); };
  v += both(dpp_move_i<0xB1>(__double2loint(v)), dpp_move_i<0xB1>(__double2hiint(v)));
  v += both(dpp_move_i<0x4E>(__double2loint(v)), dpp_move_i<0x4E>(__double2hiint(v)));
  v += both(dpp_move_i<0x141>(__double2loint(v)), dpp_move_i<0x141>(__double2hiint(v)));
  v += both(dpp_move_i<0x140>(__double2loint(v)), dpp_move_i<0x140>(__double2hiint(v)));
  auto swapped = [&](auto lo, auto hi) { return both(int(lo[0]), int(hi[0])) + both(int(lo[1]), int(hi[1])); };
  {
    const uint32_t lo = uint32_t(__double2loint(v)), hi = uint32_t(__double2hiint(v));
    v = swapped(__builtin_amdgcn_permlane16_swap(lo, lo, false, false), __builtin_amdgcn_permlane16_swap(hi, hi, false, false));
  }
  const uint32_t lo = uint32_t(__double2loint(v)), hi = uint32_t(__double2hiint(v));
  return swapped(__builtin_amdgcn_permlane32_swap(lo, lo, false, false), __builtin_amdgcn_permlane32_swap(hi, hi, false, false));
}

// The common offset is reduced first, so that each lane rescales its sums once; WAVE: 64 lanes, else 16.
template <bool WAVE> __device__ __forceinline__ RowStat stat_reduce(RowStat a) {
  auto all = [](float x, auto op) { return WAVE ? wave_reduce(x, op) : row16_reduce(x, op); };
  auto add = [](float x, float y) { return x + y; };
  const float M = all(a.m, [](float x, float y) { return fmaxf(x, y); });
  const float f = (a.m == M) ? 1.f : exp2_fast((a.m - M) * kLog2e);   // also -inf on both sides
  return RowStat{M, all(a.s * f, add), all(a.sz * f, add)};
}

// Workgroup-wide merge; every thread gets the result.  NT = threads per workgroup (at most 1024).
// (Against merging pairs of states through LDS shuffles and the waves' states one after the other in every thread:
// 0.4 % of the one-pass loss call on 151936 bf16 logits a row.)
template <int NT>
__device__ __forceinline__ RowStat stat_block_reduce(RowStat a, RowStat* lds /*[NT/64]*/) {
  a = stat_reduce<true>(a);
  constexpr int kWaves = NT / kWave;
  static_assert(kWaves <= 16, "one lane per wave in the second step");
  if constexpr (kWaves > 1) {
    const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
    if (lane == 0) lds[wave] = a;
    __syncthreads();
    a = stat_reduce<false>(lane % 16 < kWaves ? lds[lane % 16] : stat_identity());
  }
  return a;
}

// What rounding left off a log-prob; nothing where the log-prob itself is infinite (a sampled token at -inf), whose
// remainder is formed as inf - inf.
__device__ __forceinline__ float remainder_of(float lp, float low) { return fabsf(lp) < INFINITY ? low : 0.f; }

// a + b as the rounded sum and what the rounding left off (Knuth's two-sum).
struct Split {
  float sum, rest;
};
__device__ __forceinline__ Split two_sum(float a, float b) {
  const float s = a + b, bb = s - a;
  return Split{s, (a - (s - bb)) + (b - bb)};
}

// What a row's state says about its sampled token: log-partition, log-prob, and what rounding the log-prob to 32
// bits left off (for the ratio of the loss, whose terms cancel inside a group).  log s = k log 2 + log f with f in
// [1/sqrt 2, sqrt 2): k times the leading bits of log 2 (355/512, Cody and Waite's split) is exact, and the rest stays
// below 0.36 whatever s is, so that its rounding is 1.5e-8 at most and only the results are rounded at their own size.
struct RowLogProb {
  float lse, lp, low;
};
__device__ __forceinline__ RowLogProb row_logprob(const RowStat& st, float zy) {
  constexpr float kLn2Hi = 0.693359375f, kLn2Lo = -2.12194440e-4f;
  float f = __builtin_amdgcn_frexp_mantf(st.s);   // [1/2, 1)
  int k = __builtin_amdgcn_frexp_expf(st.s);
  if (f < 0.70710678f) {
    f *= 2.f;
    --k;
  }
  const float hi = float(k) * kLn2Hi, lo = fmaf(float(k), kLn2Lo, logf(f));
  const Split sum = two_sum(st.m, hi);
  const float lse = sum.sum + (sum.rest + lo);
  const float d = zy - st.m;            // an exact difference of stored values, unless they are 32-bit
  const Split a = two_sum(d, -hi);
  const Split b = two_sum(a.sum, a.rest - lo);
  if (!(fabsf(d) < INFINITY)) return RowLogProb{lse, d - (hi + lo), 0.f};   // a sampled token at -inf: no remainders
  return RowLogProb{lse, b.sum, b.rest};
}

// Loss term, its derivative with respect to the log-prob and the clip decision of one token whose rollout has
// weight w != 0 (Eq. 2; the KL term in its per-token form exp(d) - d - 1, d = log pi_ref - log pi).  flag:
// 0 = no advantage, 1 = unclipped, 2 = clipped.  ref is looked at only with kl_coef != 0.
struct LossHyper {
  float eps_lo, eps_hi, grad_scale, ent_coef, kl_coef;
};
struct TokenTerm {
  float g, term;
  int flag;
};
__device__ __forceinline__ TokenTerm token_term(const LossHyper& h, float A, float w, float lp, float low, float old_lp,
                                                float ref) {
  TokenTerm r{0.f, 0.f, 0};
  if (A != 0.f) {
    const float rho = expf(lp - old_lp + low);
    const float lo = 1.f - h.eps_lo, hi = 1.f + h.eps_hi;
    const float clipped = fminf(fmaxf(rho, lo), hi);
    const float s = fminf(rho * A, clipped * A);
    const bool unclipped = A > 0.f ? (rho <= hi) : (rho >= lo);
    r.term = -w * s;
    r.g = unclipped ? -h.grad_scale * w * A * rho : 0.f;
    r.flag = unclipped ? 1 : 2;
  }
  if (h.kl_coef != 0.f) {
    const float d = ref - lp - low;
    const float ed = expf(d);
    r.term += h.kl_coef * w * (ed - d - 1.f);
    r.g += h.grad_scale * h.kl_coef * w * (1.f - ed);
  }
  return r;
}

// Loss and clip fraction (either may be null) from T per-token terms by one workgroup of NT threads: fixed order, 64-bit sums, so that the
// result does not depend on scheduling.  Latency bound: eight tokens' loads in flight per thread (one at a time: 7.6 us at
// 16384 tokens), then two steps inside the waves and one exchange between them (a tree over LDS with a barrier per
// level: 2.8 us for 2048 tokens, 2.2 this way).
template <int NT>
__device__ __forceinline__ void loss_reduce(const float* __restrict__ term, const int32_t* __restrict__ flag, int64_t T,
                                            float* __restrict__ loss, float* __restrict__ clip_frac) {
  constexpr int kAhead = 8, kWaves = NT / kWave;
  static_assert(kWaves <= kWave, "one lane per wave in the second step");
  __shared__ double s_sum[kWaves];
  __shared__ int s_sig[kWaves], s_clip[kWaves];
  double acc = 0.0;
  int nsig = 0, nclip = 0;
  for (int64_t t0 = threadIdx.x; t0 < T; t0 += kAhead * NT) {
    float x[kAhead];
    int f[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      const int64_t t = t0 + int64_t(u) * NT;
      x[u] = t < T ? term[t] : 0.f;
      f[u] = t < T ? flag[t] : 0;
    }
#pragma unroll
    for (int u = 0; u < kAhead; ++u) {
      acc += double(x[u]);
      nsig += f[u] != 0;
      nclip += f[u] == 2;
    }
  }
  acc = wave_sum_d(acc);
  nsig = wave_sum_i(nsig);
  nclip = wave_sum_i(nclip);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  if (lane == 0) {
    s_sum[wave] = acc;
    s_sig[wave] = nsig;
    s_clip[wave] = nclip;
  }
  __syncthreads();
  if (wave != 0) return;
  acc = wave_sum_d(lane < kWaves ? s_sum[lane] : 0.0);
  nsig = wave_sum_i(lane < kWaves ? s_sig[lane] : 0);
  nclip = wave_sum_i(lane < kWaves ? s_clip[lane] : 0);
  if (lane == 0) {
    if (loss) loss[0] = float(acc);
    if (clip_frac) clip_frac[0] = nsig ? float(nclip) / float(nsig) : 0.f;
  }
}

// Fold N logits into a thread's running state.  The offset m is only moved when a value
// exceeds it by more than kLazy nats, so the rescale is rare and exp(z - m) stays below
// e^kLazy; sums of 2^24 such terms stay far inside fp32 range.
constexpr float kLazy = 12.0f;

template <int N>
__device__ __forceinline__ void stat_update(RowStat& st, const float (&z)[N]) {
  float vm = z[0];
  if constexpr (N >= 3) {
#pragma unroll
    for (int k = 1; k + 1 < N; k += 2) vm = max3(vm, z[k], z[k + 1]);
    if constexpr (N % 2 == 0) vm = fmaxf(vm, z[N - 1]);
  } else if constexpr (N == 2) {
    vm = fmaxf(vm, z[1]);
  }
  // also taken on first use (m = -inf).  The wave-uniform test in front keeps the compiler from
  // turning the rare rescale into always-executed predicated code (about two extra vector
  // instructions per logit in kernels whose vector ALUs are close to saturated).
  const bool grow = vm > st.m + kLazy;
  if (__builtin_amdgcn_ballot_w64(grow) != 0) {
    asm volatile("" ::: "memory");   // a side effect: the block cannot be if-converted
    if (grow) {
      float f = (st.m == -INFINITY) ? 0.f : exp2_fast((st.m - vm) * kLog2e);
      st.s *= f;
      st.sz *= f;
      st.m = vm;
    }
  }
  const float c = -st.m * kLog2e;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    float e = exp2_fast(fmaf(z[k], kLog2e, c));
    st.s += e;
    st.sz = fmaf(e, z[k], st.sz);
  }
}

__device__ __forceinline__ void unpack8(const u32x4_t& v, float (&z)[8]) {
  z[0] = bf16_lo(v.x); z[1] = bf16_hi(v.x);
  z[2] = bf16_lo(v.y); z[3] = bf16_hi(v.y);
  z[4] = bf16_lo(v.z); z[5] = bf16_hi(v.z);
  z[6] = bf16_lo(v.w); z[7] = bf16_hi(v.w);
}

__device__ __forceinline__ void unpack8_f16(const u32x4_t& v, float (&z)[8]) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    f16x2_t h;
    __builtin_memcpy(&h, &w[k], 4);
    z[2 * k] = float(h.x);
    z[2 * k + 1] = float(h.y);
  }
}

__device__ __forceinline__ void unpack16_f8(const u32x4_t& v, float (&z)[16]) {
  const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const f32x2_t lo = __builtin_amdgcn_cvt_pk_f32_fp8(int(w[k]), false);
    const f32x2_t hi = __builtin_amdgcn_cvt_pk_f32_fp8(int(w[k]), true);
    z[4 * k] = lo.x; z[4 * k + 1] = lo.y;
    z[4 * k + 2] = hi.x; z[4 * k + 3] = hi.y;
  }
}

// One 16-byte vector of stored logits -> floats (16 for the 8-bit type, 8 for the 2-byte types, 4 for fp32) and back.
template <int DT> __device__ __forceinline__ void unpack_vec(const u32x4_t& v, float (&z)[Storage<DT>::kPerVec]) {
  if constexpr (DT == kBF16) unpack8(v, z);
  else if constexpr (DT == kF16) unpack8_f16(v, z);
  else if constexpr (DT == kF8) unpack16_f8(v, z);
  else {
    z[0] = __uint_as_float(v.x); z[1] = __uint_as_float(v.y);
    z[2] = __uint_as_float(v.z); z[3] = __uint_as_float(v.w);
  }
}
template <int DT> __device__ __forceinline__ u32x4_t pack_vec(const float (&d)[Storage<DT>::kPerVec]) {
  u32x4_t o;
  if constexpr (DT == kBF16) {
    o.x = pack_bf16x2(d[0], d[1]); o.y = pack_bf16x2(d[2], d[3]);
    o.z = pack_bf16x2(d[4], d[5]); o.w = pack_bf16x2(d[6], d[7]);
  } else if constexpr (DT == kF16) {
    o.x = pack_f16x2(d[0], d[1]); o.y = pack_f16x2(d[2], d[3]);
    o.z = pack_f16x2(d[4], d[5]); o.w = pack_f16x2(d[6], d[7]);
  } else if constexpr (DT == kF8) {
    o.x = pack_f8x4(d[0], d[1], d[2], d[3]);     o.y = pack_f8x4(d[4], d[5], d[6], d[7]);
    o.z = pack_f8x4(d[8], d[9], d[10], d[11]);   o.w = pack_f8x4(d[12], d[13], d[14], d[15]);
  } else {
    o.x = __float_as_uint(d[0]); o.y = __float_as_uint(d[1]);
    o.z = __float_as_uint(d[2]); o.w = __float_as_uint(d[3]);
  }
  return o;
}

// A row as 16-byte aligned vectors: `head` elements in front of the first one, nvec vectors, and fewer than a
// vector's worth behind.  Rows of a tensor whose pitch is not a multiple of 16 bytes differ in head, and
// a kernel that reads logits and writes dlogits requires the two to agree in it (rows_alike).
struct RowGeom {
  int head, nvec;
};
template <int DT>
__device__ __forceinline__ RowGeom row_geom(const void* base, int64_t t, int64_t ld, int V) {
  constexpr int E = Storage<DT>::kPerVec;
  const uint32_t first = uint32_t(reinterpret_cast<uintptr_t>(base) / Storage<DT>::kBytes) + uint32_t(t * ld);
  const int head = min(int((E - first % E) % E), V);
  return RowGeom{head, (V - head) / E};
}
// The element outside the vectors that this thread looks after, -1: none.  Threads 0 .. E-1 take the head,
// E .. 2E-1 what is behind the last vector.
template <int DT>
__device__ __forceinline__ int ragged_elt(RowGeom r, int V, int tid) {
  constexpr int E = Storage<DT>::kPerVec;
  if (tid < E) return tid < r.head ? tid : -1;
  const int j = r.head + r.nvec * E + tid - E;
  return tid < 2 * E && j < V ? j : -1;
}
template <int DT> __device__ __forceinline__ char* row_ptr(const void* base, int64_t t, int64_t ld, int j = 0) {
  return const_cast<char*>(reinterpret_cast<const char*>(base)) + (size_t(t) * size_t(ld) + size_t(j)) * Storage<DT>::kBytes;
}
// Host side of the same: element-aligned logits, and a gradient (nullable) at the same offset from 16 bytes.
inline bool rows_alike(const void* logits, const void* dlogits, size_t elt) {
  const uintptr_t z = reinterpret_cast<uintptr_t>(logits), d = reinterpret_cast<uintptr_t>(dlogits);
  return z % elt == 0 && (!dlogits || z % 16 == d % 16);
}

// A launch has fewer than 2^32 threads in all (and fewer than 2^31 workgroups).
inline bool grid_fits(int64_t blocks, int threads) { return blocks < (int64_t(1) << 31) && blocks * threads < (int64_t(1) << 32); }

// Compute units of the current device (256 where it cannot be asked).
inline int compute_units() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  return hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0 ? n : 256;
}

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

inline aero_status launch_status() {
  return hipGetLastError() == hipSuccess ? AERO_OK : AERO_ERR_HIP;
}

}  // namespace aero
