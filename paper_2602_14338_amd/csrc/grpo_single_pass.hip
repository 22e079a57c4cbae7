// Forward statistics, clipped loss terms and dlogits of one token row in a single pass over
// HBM (softmax policy of App. C, surrogate of Eq. 2, gradient of App. A.1): the row is read once
// into registers (and LDS where it is long: 20 x 16 bytes per thread of 1024 at V = 151936 in bf16),
// the log-partition is reduced across the workgroup, and the gradient row is produced from the
// copy on chip - twice the row's bytes of traffic instead of three times for a forward pass followed
// by a backward pass.  All storage types, any row length up to 20 x 1024 vectors (up to four times that with what the chip does
// not hold read again), any row alignment.
#include <mutex>

#include "aero_device.h"

namespace aero {

constexpr int kSpNT = 1024;

template <int DT>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_vectors(const void* base, int64_t t, int64_t ld, RowGeom r) {
  return __builtin_amdgcn_make_buffer_rsrc(row_ptr<DT>(base, t, ld, r.head), 0, r.nvec * 16, 0x00020000);
}

// One vector of the gradient row: dz_j = pi_j (a z_j + b) + g 1[j = y]; without the entropy bonus a = 0, b = -g.
// own: the vector holds the sampled token, as its element ye.
template <int DT, bool ENT>
__device__ __forceinline__ u32x4_t grad_vec(const u32x4_t& src, float a, float b, float c, float g, bool own, int ye) {
  constexpr int E = Storage<DT>::kPerVec;
  float z[E], d[E];
  unpack_vec<DT>(src, z);
#pragma unroll
  for (int e = 0; e < E; ++e) d[e] = (ENT ? fmaf(a, z[e], b) : b) * exp2_fast(fmaf(z[e], kLog2e, c));
  if (own) {
#pragma unroll
    for (int e = 0; e < E; ++e) d[e] += (e == ye) ? g : 0.f;
  }
  return pack_vec<DT>(d);
}

// One workgroup per row, NV vectors of 16 bytes per thread in registers.
// ENT: the optional terms are on: the entropy bonus (loss and gradient row) and / or the KL penalty
// (a per-token scalar added to the loss term and to g); either coefficient may be 0.
template <int DT, int NT, int NV, bool ENT>
__global__ __launch_bounds__(NT) void k_row_single_pass(
    const void* logits, int64_t T, int V, int64_t ld, const int32_t* __restrict__ targets,
    const float* __restrict__ old_logprob, const int32_t* __restrict__ token_rollout,
    const float* __restrict__ adv, const float* __restrict__ weight, int R, float eps_lo, float eps_hi,
    float grad_scale, float ent_coef, float kl_coef, const float* __restrict__ ref_logprob, int stats_all,
    float* __restrict__ g_out, float* __restrict__ term_out,
    int32_t* __restrict__ flag_out, float* __restrict__ logprob_out, float* __restrict__ entropy_out,
    float* __restrict__ lse_out, void* dlogits, int32_t* __restrict__ err_flag) {
  __shared__ RowStat lds[NT / kWave];
  constexpr int E = Storage<DT>::kPerVec;
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x;
  const int i = token_rollout[t];
  const int y = targets[t];
  const bool valid = i >= 0 && i < R && y >= 0 && y < V;
  float A = 0.f, w = 0.f;
  if (valid) {
    A = adv[i];
    w = weight[i];
  }
  const bool signal = valid && A != 0.f && w != 0.f;
  const bool bonus = ENT && valid && w != 0.f;          // entropy bonus: every token of a weighted rollout
  const bool need = (valid && stats_all) || signal || bonus;   // uniform over the workgroup
  // asked for in front of the row: behind the row's reduction it is one more wait (8-12 us calls 0 to 3 %)
  const float old = old_logprob[t];
  const float ref = ENT && kl_coef != 0.f ? ref_logprob[t] : 0.f;
  const RowGeom geom = row_geom<DT>(logits, t, ld, V);
  const int nvec = geom.nvec, jr = ragged_elt<DT>(geom, V, tid);
  const char* zrow = row_ptr<DT>(logits, t, ld);
  char* drow = dlogits ? row_ptr<DT>(dlogits, t, ld) : nullptr;
  const u32x4_t zero = {0u, 0u, 0u, 0u};

  auto zero_fill = [&]() {
    if (!drow) return;
    u32x4_t* dv = reinterpret_cast<u32x4_t*>(drow + geom.head * Storage<DT>::kBytes);
    for (int k = tid; k < nvec; k += NT) __builtin_nontemporal_store(zero, dv + k);
    if (jr >= 0) store_elt<DT>(drow, jr, 0.f);
  };

  if (!need) {
    if (tid == 0) {
      // padding / ignored rows (a negative index) are not flagged, whatever their other index holds
      if (i >= 0 && y >= 0 && (i >= R || y >= V) && err_flag)
        atomicOr(err_flag, i >= R ? AERO_DERR_BAD_ROLLOUT : AERO_DERR_BAD_TARGET);
      g_out[t] = 0.f;
      term_out[t] = 0.f;
      flag_out[t] = 0;
      if (logprob_out) logprob_out[t] = 0.f;
      if (entropy_out) entropy_out[t] = 0.f;
      if (lse_out) lse_out[t] = 0.f;
    }
    if (i != AERO_ROW_UNTOUCHED) zero_fill();
    return;
  }

  // ---- the row -> registers.  Buffer loads: one 32-bit offset register instead of a 64-bit
  // pointer per vector, and the descriptor's bounds check returns zeros past the row's end
  // (validity is decided again at use).  aux = 2: non-temporal.
  const __amdgpu_buffer_rsrc_t zsrc = row_vectors<DT>(logits, t, ld, geom);
  const uint32_t voff = uint32_t(tid) * 16u;
  u32x4_t v[NV];
#pragma unroll
  for (int u = 0; u < NV; ++u)
    v[u] = __builtin_amdgcn_raw_buffer_load_b128(zsrc, voff + uint32_t(u) * (NT * 16u), 0, 2);
  const float zr = jr >= 0 ? load_elt<DT>(zrow, jr) : 0.f;
  const float zy = load_elt<DT>(zrow, y);   // read before any thread may overwrite the row in place

  RowStat st = stat_identity();
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    if (tid < nvec - u * NT) {
      float z[E];
      unpack_vec<DT>(v[u], z);
      stat_update<E>(st, z);
    }
    __builtin_amdgcn_sched_barrier(0);   // one vector at a time: keeps temporaries from piling up
  }
  if (jr >= 0) {
    float z[1] = {zr};
    stat_update<1>(st, z);
  }
  // Orders the loads of the row before the stores over it, for a gradient in place: by its barrier, and with one
  // wave (no barrier) because every lane's result needs every lane's loads.
  st = stat_block_reduce<NT>(st, lds);
  const RowLogProb own = row_logprob(st, zy);
  const float lse = own.lse, lp = own.lp;

  // ---- token terms (every thread computes the same scalars; token_term's text in place: called here it costs rows of
  // 1024 threads 4-13 % with the optional terms, 20254 fp32 logits 47.7 / 53.9 us) ----
  float g = 0.f, term = 0.f;
  int flag = 0;
  if (signal) {
    const float rho = expf(lp - old + own.low);
    const float lo = 1.f - eps_lo, hi = 1.f + eps_hi;
    const float clipped = fminf(fmaxf(rho, lo), hi);
    const float s = fminf(rho * A, clipped * A);
    const bool unclipped = A > 0.f ? (rho <= hi) : (rho >= lo);
    term = -w * s;
    g = unclipped ? -grad_scale * w * A * rho : 0.f;
    flag = unclipped ? 1 : 2;
  }
  const float ent = lse - st.sz / st.s;
  // gradient row: dz_j = pi_j (a z_j + b) + g 1[j = y]; without the entropy bonus a = 0, b = -g
  if (bonus && kl_coef != 0.f) {   // Eq. 2's beta term: exp(d) - d - 1, d = log pi_ref - log pi
    const float d = ref - lp - own.low;
    const float ed = expf(d);
    term += kl_coef * w * (ed - d - 1.f);
    g += grad_scale * kl_coef * w * (1.f - ed);
  }
  float a = 0.f, ng = -g;
  if (bonus) {
    term -= ent_coef * w * ent;
    a = grad_scale * ent_coef * w;
    ng = a * (ent - lse) - g;
  }
  if (tid == 0) {
    g_out[t] = g;
    term_out[t] = term;
    flag_out[t] = flag;
    if (logprob_out) logprob_out[t] = lp;
    if (entropy_out) entropy_out[t] = ent;
    if (lse_out) lse_out[t] = lse;
  }
  if (!drow) return;
  if (g == 0.f && a == 0.f) {
    zero_fill();
    return;
  }

  // ---- gradient row from the registers ----
  const float c = -lse * kLog2e;
  const __amdgpu_buffer_rsrc_t dsrc = row_vectors<DT>(dlogits, t, ld, geom);
  // the store offsets are formed again from an opaque copy of the lane offset; otherwise the
  // compiler keeps all NV load offsets alive across the reduction just to reuse them here
  uint32_t voff_st = voff;
  asm volatile("" : "+v"(voff_st));
  const int yvec = (y - geom.head) >> Storage<DT>::kLogPerVec, ye = (y - geom.head) & (E - 1);   // head: yvec = -1
#pragma unroll
  for (int u = 0; u < NV; ++u) {
    if (tid < nvec - u * NT)
      __builtin_amdgcn_raw_buffer_store_b128(grad_vec<DT, ENT>(v[u], a, ng, c, g, tid == yvec - u * NT, ye), dsrc,
                                             voff_st + uint32_t(u) * (NT * 16u), 0, 2);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (jr >= 0) {
    float d = (ENT ? fmaf(a, zr, ng) : ng) * exp2_fast(fmaf(zr, kLog2e, c));
    if (jr == y) d += g;
    store_elt<DT>(drow, jr, d);
  }
}

// ------------------------------------------------------------------------------------------
// Streaming variant for long rows.  One persistent 1024-thread workgroup per CU walks rows
// t = blockIdx.x, + gridDim.x, ...  The first NL vectors of every thread live in LDS, filled by
// buffer_load ... lds into wave-private slots; as soon as a slot has been turned into gradient
// and stored, the same slot is refilled with the NEXT row's vector, so the CU keeps reads in
// flight during its store phase (a workgroup of this size cannot share a CU with a second one).
// The remaining NV - NL vectors are ordinary register loads issued at the top of a row.
// Rows are handed out through a global counter (padding and zero-advantage rows cost far less
// than gradient rows, a fixed stride would leave CUs idle); a workgroup always knows its next
// row one row ahead, and leaves when the counter has passed T.  The counter indexes a row order
// in which the rows that are read come first and the rows that are only zero-filled last
// (k_row_order): the memory system then sees a read+write phase followed by a write-only
// phase instead of a mix of the two, which is worth several percent on padded batches.
// Rows marked AERO_ROW_UNTOUCHED are in neither part: their gradient row is not written, their
// scalars are zeroed by k_row_order, and this kernel never sees them.
// ------------------------------------------------------------------------------------------
struct RowInfo {
  int y;
  float A, w;
  bool valid, signal, bonus, need;
};

// every_weighted: the entropy bonus is on, rows of weighted rollouts with advantage 0 count too
__device__ __forceinline__ RowInfo row_info(int64_t t, int64_t T, int V, int R, const int32_t* targets,
                                            const int32_t* token_rollout, const float* adv, const float* weight,
                                            int stats_all, bool every_weighted) {
  RowInfo r{0, 0.f, 0.f, false, false, false, false};
  if (t >= T) return r;
  const int i = token_rollout[t];
  r.y = targets[t];
  r.valid = i >= 0 && i < R && r.y >= 0 && r.y < V;
  if (r.valid) {
    r.A = adv[i];
    r.w = weight[i];
  }
  r.signal = r.valid && r.A != 0.f && r.w != 0.f;
  r.bonus = every_weighted && r.valid && r.w != 0.f;
  r.need = r.signal || r.bonus || (r.valid && stats_all);
  return r;
}

// order[0 .. n) = rows with need, order[T - m .. T) = the m rows that are only zero-filled, each part in
// no particular order (wave-sized runs are placed by two counters: ctr[1] from the front, ctr[2]
// from the back).  The u rows marked AERO_ROW_UNTOUCHED are placed nowhere (n + m + u = T, the gap in the
// middle has u entries; ctr[3] counts them) and get their per-row scalars, all zero, here.
// Up to kOrderRows rows (ONE) one workgroup does it, which counts in LDS and presets ctr[0], so that the launch in front that clears
// the counters falls away: whole calls, two launches / one, 16 rows of 151936 bf16 logits 26.2 / 25.2 us, 200 32.4 / 30.9, 992 88.6 /
// 87.2, 1984 (fp16) 160.6 / 159.6.  It is the slower way for more rows, which one workgroup takes turn by turn: 16384 1210 / 1218.
constexpr int kOrderNT = 1024, kOrderAhead = 2;
constexpr int64_t kOrderRows = kOrderNT * kOrderAhead;
template <bool ONE>
__global__ __launch_bounds__(ONE ? kOrderNT : 256) void k_row_order(
    int64_t T, int V, int R, const int32_t* __restrict__ targets, const int32_t* __restrict__ token_rollout,
    const float* __restrict__ adv, const float* __restrict__ weight, int stats_all, int every_weighted, int first_next,
    int32_t* __restrict__ ctr, int32_t* __restrict__ order, float* __restrict__ g_out, float* __restrict__ term_out,
    int32_t* __restrict__ flag_out, float* __restrict__ logprob_out, float* __restrict__ entropy_out,
    float* __restrict__ lse_out) {
  constexpr int NT = ONE ? kOrderNT : 256, kAhead = ONE ? kOrderAhead : 1;
  __shared__ int32_t own[4];
  const int lane = threadIdx.x & 63;
  if constexpr (ONE) {
    if (threadIdx.x < 4) own[threadIdx.x] = threadIdx.x == 0 ? first_next : 0;
    __syncthreads();
  }
  int32_t* const count = ONE ? own : ctr;
  bool untouched[kAhead], need[kAhead];
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    const int64_t t = (int64_t(blockIdx.x) * kAhead + u) * NT + threadIdx.x;
    untouched[u] = t < T && token_rollout[t] == AERO_ROW_UNTOUCHED;
    need[u] = row_info(t, T, V, R, targets, token_rollout, adv, weight, stats_all, every_weighted != 0).need;
  }
#pragma unroll
  for (int u = 0; u < kAhead; ++u) {
    const int64_t t = (int64_t(blockIdx.x) * kAhead + u) * NT + threadIdx.x;
    const bool rest = t < T && !need[u] && !untouched[u];
    const uint64_t m_need = __ballot(need[u]), m_rest = __ballot(rest), m_unt = __ballot(untouched[u]);
    const uint64_t below = (uint64_t(1) << lane) - 1;
    int base_need = 0, base_rest = 0;
    if (lane == 0) {
      if (m_need) base_need = atomicAdd(count + 1, __popcll(m_need));
      if (m_rest) base_rest = atomicAdd(count + 2, __popcll(m_rest));
      if (m_unt) atomicAdd(count + 3, __popcll(m_unt));
    }
    if (untouched[u]) {
      g_out[t] = 0.f;
      term_out[t] = 0.f;
      flag_out[t] = 0;
      if (logprob_out) logprob_out[t] = 0.f;
      if (entropy_out) entropy_out[t] = 0.f;
      if (lse_out) lse_out[t] = 0.f;
    }
    base_need = __shfl(base_need, 0, kWave);
    base_rest = __shfl(base_rest, 0, kWave);
    if (need[u]) order[base_need + __popcll(m_need & below)] = int32_t(t);
    if (rest) order[T - 1 - (base_rest + __popcll(m_rest & below))] = int32_t(t);
  }
  if constexpr (ONE) {
    __syncthreads();
    if (threadIdx.x < 4) ctr[threadIdx.x] = own[threadIdx.x];
  }
}

constexpr int kTailAhead = 4;
template <int DT, int NV, int NL, bool ENT, bool LONG>
__global__ __launch_bounds__(kSpNT) void k_row_stream(
    const void* logits, int64_t T, int V, int64_t ld, const int32_t* __restrict__ targets,
    const float* __restrict__ old_logprob, const int32_t* __restrict__ token_rollout,
    const float* __restrict__ adv, const float* __restrict__ weight, int R, float eps_lo, float eps_hi,
    float grad_scale, float ent_coef, float kl_coef, const float* __restrict__ ref_logprob, int stats_all,
    float* __restrict__ g_out, float* __restrict__ term_out,
    int32_t* __restrict__ flag_out, float* __restrict__ logprob_out, float* __restrict__ entropy_out,
    float* __restrict__ lse_out, void* dlogits, int32_t* __restrict__ err_flag, int32_t* row_counter,
    const int32_t* __restrict__ order) {
  // positions 0 .. P of the hand-out skip the gap that the untouched rows leave in the row order
  const int n_front = row_counter[1];
  const int n_gap = row_counter[3];
  const int64_t P = T - n_gap;
  auto row_at = [&](int64_t p) -> int64_t { return p < P ? order[p < n_front ? p : p + n_gap] : T; };
  __shared__ RowStat lds[2][kSpNT / kWave];   // alternating: one barrier per row is enough
  __shared__ int s_next;
  extern __shared__ __align__(16) u32x4_t slots_raw[];   // NL x kSpNT vectors
  u32x4_t(*slots)[kSpNT] = reinterpret_cast<u32x4_t(*)[kSpNT]>(slots_raw);
  constexpr int NR = NV - NL;
  const int tid = threadIdx.x;
  constexpr int E = Storage<DT>::kPerVec;
  const uint32_t voff = uint32_t(tid) * 16u;
  const u32x4_t zero = {0u, 0u, 0u, 0u};
  auto dma_slot = [&](__amdgpu_buffer_rsrc_t src, int u) {   // lane l of wave w lands at slots[u][64 w + l]
    __builtin_amdgcn_raw_ptr_buffer_load_lds(src, &slots[u][(tid >> 6) << 6], 16,
                                             voff + uint32_t(u) * (kSpNT * 16u), 0, 0, 2);
  };

  // the first gridDim.x positions of the row order are assigned by workgroup id; the counter
  // starts at gridDim.x.  pn = position of the next row, tn = that row (T = none left)
  int64_t t = row_at(blockIdx.x);
  if (tid == 0) s_next = atomicAdd(row_counter, 1);
  __syncthreads();
  // uniform values read from LDS look divergent to the compiler: said explicitly, the row's pointers, descriptors
  // and scalars live in scalar registers
  int64_t pn = __builtin_amdgcn_readfirstlane(s_next);
  int64_t tn = row_at(pn);
  RowInfo cur = row_info(t, T, V, R, targets, token_rollout, adv, weight, stats_all, ENT);
  RowGeom geom = row_geom<DT>(logits, t, ld, V);
  if (cur.need) {
    const __amdgpu_buffer_rsrc_t src = row_vectors<DT>(logits, t, ld, geom);
#pragma unroll
    for (int u = 0; u < NL; ++u) dma_slot(src, u);
  }

  int reduces = 0;   // selects the LDS buffer of the next reduction
  while (t < T) {
    const RowInfo nxt = row_info(tn, T, V, R, targets, token_rollout, adv, weight, stats_all, ENT);
    const int nvec = geom.nvec, jr = ragged_elt<DT>(geom, V, tid);
    const char* zrow = row_ptr<DT>(logits, t, ld);
    char* drow = dlogits ? row_ptr<DT>(dlogits, t, ld) : nullptr;
    const RowGeom ngeom = nxt.need ? row_geom<DT>(logits, tn, ld, V) : geom;
    const __amdgpu_buffer_rsrc_t nsrc = row_vectors<DT>(logits, nxt.need ? tn : t, ld, ngeom);
    float g = 0.f, term = 0.f, lp = 0.f, ent = 0.f, lse = 0.f;
    float ea = 0.f;   // entropy bonus: grad_scale c w of this row (ENT only)
    int flag = 0;
    u32x4_t v[NR];
    float zr = 0.f;

    if (cur.need) {   // uniform over the workgroup
      const __amdgpu_buffer_rsrc_t zsrc = row_vectors<DT>(logits, t, ld, geom);
      // thread offsets are formed per row from opaque copies (and bounds compared on the scalar side): hoisted out
      // of the row loop they are forty registers, which the variants with the optional terms would spill
      uint32_t voff_ld = voff;
      asm volatile("" : "+v"(voff_ld));
#pragma unroll
      for (int u = 0; u < NR; ++u)
        v[u] = __builtin_amdgcn_raw_buffer_load_b128(zsrc, voff_ld + uint32_t(NL + u) * (kSpNT * 16u), 0, 2);
      zr = jr >= 0 ? load_elt<DT>(zrow, jr) : 0.f;
      const float zy = load_elt<DT>(zrow, cur.y);   // read before any thread may overwrite the row in place
      // Loads return in order and at least NR of them were issued just above (the sampled token's may be a scalar
      // load, which counts elsewhere): once no more than NR memory operations are outstanding, the older loads
      // into this wave's LDS slots have landed (the compiler does not track those; stores may retire in any order,
      // they only make the wait longer).
      static_assert(NR <= 15, "immediate below holds vmcnt in 4 bits");
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_waitcnt(0x0F70 | NR);
      asm volatile("" ::: "memory");
      RowStat st = stat_identity();
#pragma unroll
      for (int u = 0; u < NL; ++u) {
        if (tid < nvec - u * kSpNT) {
          const u32x4_t pv = slots[u][tid];
          float z[E];
          unpack_vec<DT>(pv, z);
          stat_update<E>(st, z);
        }
        __builtin_amdgcn_sched_barrier(0);   // one vector at a time: keeps temporaries from piling up
      }
#pragma unroll
      for (int u = 0; u < NR; ++u) {
        if (tid < nvec - (NL + u) * kSpNT) {
          float z[E];
          unpack_vec<DT>(v[u], z);
          stat_update<E>(st, z);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (LONG) {   // what the CU does not hold: plain loads, so that the memory-side cache has it for the second time
        for (int from = NV * kSpNT; from < nvec; from += kTailAhead * kSpNT) {   // uniform
          u32x4_t w[kTailAhead];
#pragma unroll
          for (int u = 0; u < kTailAhead; ++u)
            w[u] = __builtin_amdgcn_raw_buffer_load_b128(zsrc, voff_ld + uint32_t(from + u * kSpNT) * 16u, 0, 0);
#pragma unroll
          for (int u = 0; u < kTailAhead; ++u) {
            if (tid < nvec - from - u * kSpNT) {
              float z[E];
              unpack_vec<DT>(w[u], z);
              stat_update<E>(st, z);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      if (jr >= 0) {
        float z[1] = {zr};
        stat_update<1>(st, z);
      }
      st = stat_block_reduce<kSpNT>(st, lds[reduces++ & 1]);   // its barrier also orders loads before stores
      const RowLogProb own = row_logprob(st, zy);
      lse = own.lse;
      lp = own.lp;
      ent = lse - st.sz / st.s;
      if (cur.signal) {   // every thread computes the same scalars
        const float rho = expf(lp - old_logprob[t] + own.low);
        const float lo = 1.f - eps_lo, hi = 1.f + eps_hi;
        const float clipped = fminf(fmaxf(rho, lo), hi);
        const float s = fminf(rho * cur.A, clipped * cur.A);
        const bool unclipped = cur.A > 0.f ? (rho <= hi) : (rho >= lo);
        term = -cur.w * s;
        g = unclipped ? -grad_scale * cur.w * cur.A * rho : 0.f;
        flag = unclipped ? 1 : 2;
      }
      if constexpr (ENT) {
        if (cur.bonus) {
          if (kl_coef != 0.f) {   // Eq. 2's beta term: exp(d) - d - 1, d = log pi_ref - log pi
            const float d = ref_logprob[t] - lp - own.low;
            const float ed = expf(d);
            term += kl_coef * cur.w * (ed - d - 1.f);
            g += grad_scale * kl_coef * cur.w * (1.f - ed);
          }
          term -= ent_coef * cur.w * ent;
          ea = grad_scale * ent_coef * cur.w;
        }
      }
    }
    if (tid == 0) {
      if (!cur.valid && err_flag) {
        const int i = token_rollout[t];
        if (i >= 0 && cur.y >= 0 && (i >= R || cur.y >= V))   // padding / ignored rows are not flagged
          atomicOr(err_flag, i >= R ? AERO_DERR_BAD_ROLLOUT : AERO_DERR_BAD_TARGET);
      }
      g_out[t] = g;
      term_out[t] = term;
      flag_out[t] = flag;
      if (logprob_out) logprob_out[t] = lp;
      if (entropy_out) entropy_out[t] = ent;
      if (lse_out) lse_out[t] = lse;
    }

    if (drow && (g != 0.f || (ENT && ea != 0.f))) {
      const float c = -lse * kLog2e;
      // gradient row: dz_j = pi_j (a z_j + ng) + g 1[j = y]; without the entropy bonus a = 0, ng = -g
      const float a = ea;
      const float ng = ENT ? ea * (ent - lse) - g : -g;
      const __amdgpu_buffer_rsrc_t dsrc = row_vectors<DT>(dlogits, t, ld, geom);
      uint32_t voff_st = voff;
      asm volatile("" : "+v"(voff_st));
      const int y = cur.y, yvec = (y - geom.head) >> Storage<DT>::kLogPerVec, ye = (y - geom.head) & (E - 1);
#pragma unroll
      for (int u = 0; u < NL; ++u) {   // LDS part first: each slot is refilled right after its last use
        const u32x4_t pv = slots[u][tid];
        if (tid < nvec - u * kSpNT)
          __builtin_amdgcn_raw_buffer_store_b128(grad_vec<DT, ENT>(pv, a, ng, c, g, tid == yvec - u * kSpNT, ye), dsrc,
                                                 voff_st + uint32_t(u) * (kSpNT * 16u), 0, 2);
        asm volatile("" ::: "memory");
        if (nxt.need) dma_slot(nsrc, u);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int u = 0; u < NR; ++u) {
        if (tid < nvec - (NL + u) * kSpNT)
          __builtin_amdgcn_raw_buffer_store_b128(grad_vec<DT, ENT>(v[u], a, ng, c, g, tid == yvec - (NL + u) * kSpNT, ye), dsrc,
                                                 voff_st + uint32_t(NL + u) * (kSpNT * 16u), 0, 2);
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (LONG) {
        const __amdgpu_buffer_rsrc_t zsrc = row_vectors<DT>(logits, t, ld, geom);
        for (int from = NV * kSpNT; from < nvec; from += kTailAhead * kSpNT) {   // uniform
          u32x4_t w[kTailAhead];
#pragma unroll
          for (int u = 0; u < kTailAhead; ++u)
            w[u] = __builtin_amdgcn_raw_buffer_load_b128(zsrc, voff_st + uint32_t(from + u * kSpNT) * 16u, 0, 2);
#pragma unroll
          for (int u = 0; u < kTailAhead; ++u) {
            const int k = from + u * kSpNT;
            if (tid < nvec - k)
              __builtin_amdgcn_raw_buffer_store_b128(grad_vec<DT, ENT>(w[u], a, ng, c, g, tid == yvec - k, ye), dsrc,
                                                     voff_st + uint32_t(k) * 16u, 0, 2);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
      if (jr >= 0) {
        float d = (ENT ? fmaf(a, zr, ng) : ng) * exp2_fast(fmaf(zr, kLog2e, c));
        if (jr == y) d += g;
        store_elt<DT>(drow, jr, d);
      }
    } else {
      // this row's slots are no longer needed: make sure every read of them has returned
      __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
      asm volatile("" ::: "memory");
      if (nxt.need) {
#pragma unroll
        for (int u = 0; u < NL; ++u) dma_slot(nsrc, u);
      }
      if (drow) {   // zero fill
        u32x4_t* dv = reinterpret_cast<u32x4_t*>(drow + geom.head * Storage<DT>::kBytes);
        for (int k = tid; k < nvec; k += kSpNT) __builtin_nontemporal_store(zero, dv + k);
        if (jr >= 0) store_elt<DT>(drow, jr, 0.f);
      }
    }
    // hand-over: the row after the next one is drawn now (all threads have read s_next)
    __syncthreads();
    if (tid == 0) s_next = pn < P ? atomicAdd(row_counter, 1) : int(T);
    __syncthreads();
    cur = nxt;
    geom = row_geom<DT>(logits, tn, ld, V);
    t = tn;
    pn = __builtin_amdgcn_readfirstlane(s_next);
    tn = row_at(pn);
  }
}

// ctr[0]: row counter of k_row_stream (starts past the rows assigned by workgroup id),
// ctr[1], ctr[2]: fill counters of k_row_order<false>, ctr[3]: its count of untouched rows
__global__ void k_set_counter(int32_t* ctr, int32_t v) {
  ctr[0] = v;
  ctr[1] = 0;
  ctr[2] = 0;
  ctr[3] = 0;
}

constexpr int kStreamVecs = 20, kHeldVecs = 8, kLongVecs = 80;

// Threads of the workgroup that takes a row of at most kHeldVecs x 1024 vectors: the fewest that hold it in kHeldVecs
// vectors each, so that a CU works on several rows.
// (against 4 vectors each, 8192 bf16 rows: V = 3000 25.0 / 29.6 us, 6000 even, 12000 78.7 / 76.7, 24000 140 / 161, 50000 even)
inline int row_threads(int nvec) {
  return nvec <= kHeldVecs * 64 ? 64 : nvec <= kHeldVecs * 256 ? 256 : nvec <= kHeldVecs * 512 ? 512 : kSpNT;
}

// True when a single-pass kernel applies: element-aligned rows of at most 20 vectors per thread of 1024 (80, of which a CU
// holds 20 and reads the others again), and logits and dlogits alike in their position relative to 16 bytes.
//
// Where it does, it is not always the faster one; times of two passes / one pass by storage type, every row with a
// gradient:
//   up to 8 vectors per thread   a CU works on several rows: 1.1-2.5.  Loss only, 8-bit rows of more than 4096
//                                vectors: the row is held for nothing, 1.06-1.4 up to 512 rows, 0.65-0.98 from 600 on
//   more (streaming)             a row takes a CU of its own.
//     loss only                  0.55-1.0
//     T <= 256, all at once      two passes spread the gradient of a few rows over the CUs, and the more logits a vector
//                                holds, the longer a lone CU takes: fp32 1.0-1.4 from one row on, fp16 0.8-1.1 up to 32
//                                rows and 1.03-1.25 from 96 on, 8-bit 0.7-1.05 up to 160 and 1.02-1.12 from 200 on
//     more rows                  up to 320 MB, which the 256 MB memory-side cache holds for the second pass, 0.8-1.05;
//                                beyond fp16 1.00-1.17, fp32 1.06-1.19, 8-bit 0.92-1.13
//   over 20 vectors per thread   the CU holds 20 and reads the rest again, from the memory-side cache: 4 to 6 bytes per 2-byte
//                                logit instead of 6.  With a gradient in every row / right-padded, 9 of 16 rows valid:
//     up to 256 rows             the longer a 16-bit row, the more of them it takes, one per 6 KB: V = 170000 64 rows 0.98 / 0.95, 96 1.06 / 0.94, 128
//                                1.13 / 0.93, 256 1.14 / 1.04; 262144 64 rows 0.99 / 0.91, 96 1.05 / 0.93, 128 1.11 / 0.93; 400000 64 rows
//                                0.95 / 0.87, 96 0.99 / 0.89, 128 1.08 / 0.95, 256 1.27 / 1.14; 650000 96 rows 0.93 / 0.86, 128 1.0 / 0.89, 192
//                                1.18 / 1.02.  fp32 from 24 rows and 10 MB on 0.95-1.25 / 1.0-1.2 (24 of 90000 0.82 / 1.01, of 164000
//                                1.13 / 1.18; over 64 vectors per thread 96 rows 0.97 / 0.93, 256 1.19 / 1.18).  8-bit 192 rows 0.97-1.1 / 0.82-0.93, 256 1.04-1.16 / 0.85-0.95
//     more, up to 256 MB         two passes find the rows in that cache and one starts a second round of rows: 0.78-1.03 / 0.91-1.28
//     beyond                     1.0-1.4 / 1.0-1.5 (V = 262144: bf16 3072 rows 670 / 534 us, fp32 1536 667 / 560; V = 600000, 8-bit 2688
//                                rows 798 / 614)
// For held rows, more than 256 of them take the one pass for the batches that the call is for, where padding and rollouts without advantage cost the
// one pass least (9 of 16 rows valid, a third of the groups all equal: fp16 1.19-1.42, fp32 1.4-2.0, 8-bit 1.09-1.27;
// packed: fp16 0.99-1.34, 8-bit 0.87-1.23).  Held bf16 rows take it throughout: streaming 0.76-1.08 up to 8 rows,
// 0.84-1.3 from 64 on, loss only 0.55-0.99.
bool single_pass_applicable(int32_t dtype, int64_t T, int V, const void* logits, const void* dlogits) {
  const size_t elt = storage_bytes(dtype);
  const size_t nvec = size_t(V) * elt / 16;
  if (nvec > size_t(kLongVecs) * kSpNT || !rows_alike(logits, dlogits, elt)) return false;
  if (nvec <= size_t(kHeldVecs) * kSpNT && !grid_fits(T, row_threads(int(nvec)))) return false;
  if (nvec > size_t(kStreamVecs) * kSpNT) {
    if (!dlogits) return false;
    if (size_t(T) * nvec * 16 >= (size_t(256) << 20)) return true;
    if (T > 256 || dtype == AERO_F8E4M3) return false;
    return dtype == AERO_F32 ? T >= 24 && size_t(T) * nvec >= 640 * kSpNT : T >= int64_t(nvec / 384);
  }
  if (dtype == AERO_BF16) return true;
  if (nvec <= size_t(kHeldVecs) * kSpNT) return dlogits || dtype != AERO_F8E4M3 || nvec <= 4 * kSpNT || T <= 512;
  if (!dlogits) return false;
  return T >= (dtype == AERO_F32 ? 1 : dtype == AERO_F16 ? 96 : 192);
}

struct RowArgs {
  const void* logits;
  int64_t T;
  int V;
  int64_t ld;
  const int32_t* targets;
  const float* old_logprob;
  const int32_t* token_rollout;
  const float *adv, *weight;
  int R;
  float eps_lo, eps_hi, grad_scale, ent_coef, kl_coef;
  const float* ref_logprob;
  int stats_all;
  float *g, *term;
  int32_t* flag;
  float *logprob_out, *entropy_out, *lse_out;
  void* dlogits;
  int32_t* err_flag;
};

template <int DT, int NT, bool ENT>
static void launch_rows(const RowArgs& r, hipStream_t s) {
  hipLaunchKernelGGL((k_row_single_pass<DT, NT, kHeldVecs, ENT>), dim3(unsigned(r.T)), dim3(NT), 0, s, r.logits, r.T, r.V, r.ld,
                     r.targets, r.old_logprob, r.token_rollout, r.adv, r.weight, r.R, r.eps_lo, r.eps_hi, r.grad_scale,
                     r.ent_coef, r.kl_coef, r.ref_logprob, r.stats_all, r.g, r.term, r.flag, r.logprob_out,
                     r.entropy_out, r.lse_out, r.dlogits, r.err_flag);
}

template <int DT, bool ENT>
static aero_status single_pass_launch_t(const RowArgs& r, int32_t* row_counter, int32_t* row_order, hipStream_t s) {
  const int nvec = r.V / Storage<DT>::kPerVec;
  if (nvec <= kHeldVecs * kSpNT) {
    switch (row_threads(nvec)) {
      case 64: launch_rows<DT, 64, ENT>(r, s); break;
      case 256: launch_rows<DT, 256, ENT>(r, s); break;
      case 512: launch_rows<DT, 512, ENT>(r, s); break;
      default: launch_rows<DT, kSpNT, ENT>(r, s);
    }
  } else {
    constexpr int NL = 9;
    constexpr int kLdsBytes = NL * kSpNT * 16;   // 144 KB of wave-private slots
    // raising the dynamic-LDS limit is per function; done once per process, safely from any thread
    static std::once_flag attr_once;
    static hipError_t attr_rc = hipSuccess;
    std::call_once(attr_once, [&] {
      const void* const kernels[] = {reinterpret_cast<const void*>(k_row_stream<DT, kStreamVecs, NL, ENT, false>),
                                     reinterpret_cast<const void*>(k_row_stream<DT, kStreamVecs, NL, ENT, true>)};
      for (const void* k : kernels) {
        const hipError_t rc = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
        if (rc != hipSuccess) attr_rc = rc;
      }
    });
    if (attr_rc != hipSuccess) return AERO_ERR_HIP;
    const auto kernel = nvec <= kStreamVecs * kSpNT ? k_row_stream<DT, kStreamVecs, NL, ENT, false>
                                                    : k_row_stream<DT, kStreamVecs, NL, ENT, true>;
    const int cus = compute_units();
    const unsigned grid = unsigned(r.T < cus ? r.T : cus);   // one persistent workgroup per CU
    const bool one = r.T <= kOrderRows;
    if (!one) hipLaunchKernelGGL(k_set_counter, dim3(1), dim3(1), 0, s, row_counter, int32_t(grid));
    const auto order = one ? k_row_order<true> : k_row_order<false>;
    hipLaunchKernelGGL(order, dim3(one ? 1u : unsigned((r.T + 255) / 256)), dim3(one ? kOrderNT : 256), 0, s, r.T, r.V, r.R, r.targets,
                       r.token_rollout, r.adv, r.weight, r.stats_all, ENT ? 1 : 0, int(grid), row_counter, row_order, r.g, r.term,
                       r.flag, r.logprob_out, r.entropy_out, r.lse_out);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSpNT), kLdsBytes, s, r.logits, r.T, r.V, r.ld, r.targets,
                       r.old_logprob, r.token_rollout, r.adv, r.weight, r.R, r.eps_lo, r.eps_hi, r.grad_scale, r.ent_coef,
                       r.kl_coef, r.ref_logprob, r.stats_all, r.g, r.term, r.flag, r.logprob_out, r.entropy_out, r.lse_out,
                       r.dlogits, r.err_flag, row_counter, row_order);
  }
  return AERO_OK;
}

template <int DT>
static aero_status single_pass_launch_dt(const RowArgs& r, int32_t* row_counter, int32_t* row_order, hipStream_t s) {
  // a non-zero entropy or KL coefficient selects the kernels that carry the optional terms
  return r.ent_coef != 0.f || r.kl_coef != 0.f ? single_pass_launch_t<DT, true>(r, row_counter, row_order, s)
                                               : single_pass_launch_t<DT, false>(r, row_counter, row_order, s);
}

aero_status single_pass_launch(const void* logits, int32_t dtype, int64_t T, int V, int64_t ld, const int32_t* targets,
                               const float* old_logprob, const int32_t* token_rollout, const float* adv,
                               const float* weight, int R, float eps_lo, float eps_hi, float grad_scale,
                               float ent_coef, float kl_coef, const float* ref_logprob, int stats_all, float* g,
                               float* term, int32_t* flag, float* logprob_out, float* entropy_out, float* lse_out,
                               void* dlogits, int32_t* err_flag, int32_t* row_counter, int32_t* row_order,
                               hipStream_t s) {
  const RowArgs r{logits, T, V, ld, targets, old_logprob, token_rollout, adv, weight, R, eps_lo, eps_hi, grad_scale,
                  ent_coef, kl_coef, ref_logprob, stats_all, g, term, flag, logprob_out, entropy_out, lse_out, dlogits,
                  err_flag};
  switch (dtype) {
    case AERO_BF16: return single_pass_launch_dt<kBF16>(r, row_counter, row_order, s);
    case AERO_F16: return single_pass_launch_dt<kF16>(r, row_counter, row_order, s);
    case AERO_F8E4M3: return single_pass_launch_dt<kF8>(r, row_counter, row_order, s);
    default: return single_pass_launch_dt<kF32>(r, row_counter, row_order, s);
  }
}

}  // namespace aero
