// Capacity-aware evaluation of few candidate deployments over windows of a few to a few hundred requests.
//
// With few candidates the chip is mostly idle, and what counts is how long one window takes after the
// other.  A block owns a candidate: thread j keeps instance j (state, profile evaluation, the drain between
// windows), a few neighbouring lanes share a request and walk the instances in LDS between them.  Looking
// for the instances that matter first, as sweep_window_kernel does, would itself be the longest part of
// such a window: a step for each that stays, sixteen where most differ.
//
// What bounds it: a chain of two barriers, the profile rows, the walk and the sums per window.  8 candidates,
// us per window, as sweep_window_kernel or sweep_seq_kernel takes it against this one: 16 slots, windows of 9:
// 3.45 / 1.40, of 128: 1.89 / 1.37; 64 slots, of 33: 4.41 / 1.92, of 256: 4.25 / 3.82; 256 slots, all different, of
// 17: 16.2 / 2.7, of 128: 14.3 / 6.3.
//
// The arithmetic is the windowed kernel's, operation by operation.
#pragma once

#include "sweep_window_kernels.hpp"

#pragma clang fp contract(off)

namespace maaso {

// Arg-max of (slack, index) over 2^log2 consecutive lanes, at most 16, lowest index among equal slacks (see
// argmax_lanes).
__device__ __forceinline__ void argmax_group(float& s, int32_t& i, uint32_t log2) {
  if (log2 == 0u) return;
  float m = s;
  MAASO_DPP_FOLD("v_max_f32_dpp", m, "quad_perm:[1,0,3,2]");
  if (log2 >= 2u) MAASO_DPP_FOLD("v_max_f32_dpp", m, "quad_perm:[2,3,0,1]");
  if (log2 >= 3u) MAASO_DPP_FOLD("v_max_f32_dpp", m, "row_half_mirror");
  if (log2 >= 4u) MAASO_DPP_FOLD("v_max_f32_dpp", m, "row_mirror");
  uint32_t c = (s == m) ? (uint32_t)i : 0xffffffffu;
  MAASO_DPP_FOLD("v_min_u32_dpp", c, "quad_perm:[1,0,3,2]");
  if (log2 >= 2u) MAASO_DPP_FOLD("v_min_u32_dpp", c, "quad_perm:[2,3,0,1]");
  if (log2 >= 3u) MAASO_DPP_FOLD("v_min_u32_dpp", c, "row_half_mirror");
  if (log2 >= 4u) MAASO_DPP_FOLD("v_min_u32_dpp", c, "row_mirror");
  i = (int32_t)c;
  s = m;
}

// kSQ: the distributor's shortest-queue rule instead of the largest slack.  2^lpr_log2 lanes per request.
constexpr int kBlockThreads = 256;  // one per instance slot
constexpr uint32_t kBlockTrip = 4;  // records a lane reads ahead of their use
constexpr uint32_t kMaxLprLog2 = 4;
template <bool kScore, bool kSQ>
__global__ __launch_bounds__(kBlockThreads) void sweep_block_kernel(const SweepWindowArgs a, uint32_t lpr_log2) {
  constexpr uint32_t T = kBlockThreads;
  constexpr uint32_t U = kBlockTrip;
  constexpr uint32_t kPad = U << kMaxLprLog2;  // records are padded to whole trips
  const uint32_t lpr = 1u << lpr_log2, step = U << lpr_log2;
  extern __shared__ __align__(16) unsigned char smem[];
  float* tab = reinterpret_cast<float*>(smem);
  __shared__ float4 recs[256 + kPad];
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ uint32_t n_sum[256];
  __shared__ unsigned long long t_sum[256];
  __shared__ int32_t occ_s[kSQ ? 256 : 1];
  __shared__ float rank_s[kSQ ? 256 + kPad : 1];
  __shared__ uint32_t sat_part[T / 64u];
  __shared__ unsigned long long wait_part[T / 64u];

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t set = blockIdx.x / a.n_cand;
  const uint32_t c = blockIdx.x - set * a.n_cand;
  const SweepWindowSet rs = resolve_set(a.sets[set]);
  const size_t base = (size_t)c * a.i_pad;
  const uint32_t n = min(a.n_inst[c], a.i_pad);
  const bool mine = tid < n;
  LiveSlot slot;
  slot.clear();
  if (mine) slot.load(a.mp, a.tp_idx[base + tid], a.max_batch[base + tid], a.occ[base + tid], a.q_ticks[base + tid]);
  if (tid < a.n_slo) cls[tid] = ClassRow{a.d_ttft[tid], a.d_tbt[tid], a.i_ttft[tid], a.i_tbt[tid]};
  for (uint32_t i = tid; i < 3u * a.cells; i += T) tab[i] = a.tab[i];
  for (uint32_t i = tid; i < 256u + kPad; i += T) recs[i] = make_float4(1.0f, 1.0f, 1.0f, INFINITY);  // never chosen
  __syncthreads();

  const uint32_t R = rs.n_req;
  auto window_end = [&](uint32_t s0) __attribute__((always_inline)) { return R - s0 > rs.window ? s0 + rs.window : R; };
  const uint32_t per_pass = T >> lpr_log2, part = tid & (lpr - 1u), in_pass = tid >> lpr_log2;
  uint32_t sat = 0;                    // of this thread's instance
  unsigned long long wait_sum = 0ull;  // queue waits of its requests, in ticks
  float inv_tbt_first = 0.0f;
  unsigned long long bad_slot = 0ull;

  // a window's first requests are fetched a window ahead and prepared behind its predecessor
  RequestRaw raw = fetch_request(rs, 0u, in_pass, window_end(0u));
  RequestSide first = request_side(raw, a.n_slo, cls, a.status);
  uint32_t t_begin = 0, t_end = 0;
  if (R > rs.window) { t_begin = rs.arrival_ticks[0]; t_end = rs.arrival_ticks[rs.window]; }

  for (uint32_t s0 = 0, e0 = 0; s0 < R; s0 = e0) {
    e0 = window_end(s0);
    SlotRecord rec;
    float svc;
    unsigned long long bad;
    // (kPinned, 37 to 900 candidates, windows of 8 to 200, largest slack: scores of 3 to 8 slots 0.97 to 0.98 of the time, sweeps 1.02 to 1.03)
    slot.template stage<kScore>(tab, a.cells, a.mp, rec, svc, bad);
    bad_slot |= bad;  // (a thread without an instance is never bad)
    if (kScore && s0 == 0u) inv_tbt_first = in_mask(bad) ? 0.0f : 1.0f / rec.tbt;
    if (mine) {
      recs[tid] = make_float4(rec.a, rec.p, rec.tbt, rec.wait);
      n_sum[tid] = 0u;
      t_sum[tid] = 0ull;
      if (kSQ) occ_s[tid] = slot.occ;
    }
    uint32_t t_next = 0;
    raw = RequestRaw{0u, 0u, kNoRequest};
    if (e0 < R) {
      raw = fetch_request(rs, e0, in_pass, window_end(e0));
      if (window_end(e0) < R) t_next = rs.arrival_ticks[window_end(e0)];
    }
    __syncthreads();
    if (kSQ) {
      if (mine) rank_s[tid] = queue_rank_value(occ_s, n, tid);
      __syncthreads();
    }
    for (uint32_t b0 = s0; b0 < e0; b0 = e0 - b0 > per_pass ? b0 + per_pass : e0) {
      RequestSide q = first;
      if (b0 != s0) q = request_side(fetch_request(rs, b0, in_pass, e0), a.n_slo, cls, a.status);
      const Deadlines d{q.u.y, q.u.z, q.w.z, q.w.x, q.w.y, q.w.w};
      float best = -INFINITY;
      int32_t idx = -1;
      for (uint32_t j = part; j < n; j += step) {
        float4 r[U];
        float rank[U];
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          r[u] = recs[j + u * lpr];
          rank[u] = kSQ ? rank_s[j + u * lpr] : 0.0f;
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          const float slack = score_triple(r[u].x, r[u].y, r[u].z, r[u].w, q.u.x, q.u.w, d).slack;
          const float val = (kSQ && slack >= 0.0f) ? rank[u] : slack;
          idx = val > best ? (int32_t)(j + u * lpr) : idx;
          best = max_no_nan(best, val);
        }
      }
      argmax_group(best, idx, lpr_log2);
      const bool adm = best >= 0.0f && part == 0u;  // admitted requests load their instance
      const unsigned long long am = lane_mask(adm);
      if (am == 0ull) continue;
      const float4 w = recs[adm ? idx : 0];
      const unsigned long long ticks = adm ? to_ticks(fmaf(w.y, q.u.x, w.x), a.bounds.narrow) : 0ull;
      const int32_t one = __builtin_amdgcn_readlane(idx, (int)__builtin_ctzll(am));
      if (lane_mask(adm && idx == one) == am) {  // the whole wavefront chose one instance
        const unsigned long long sum = wave_sum_ticks(ticks);
        if (lane == 0u) {
          atomicAdd(&n_sum[one], (uint32_t)__popcll(am));
          atomicAdd(&t_sum[one], sum);
        }
      } else if (adm) {
        atomicAdd(&n_sum[idx], 1u);
        atomicAdd(&t_sum[idx], ticks);
      }
    }
    first = request_side(raw, a.n_slo, cls, a.status);
    lds_atomics_barrier();
    if (mine) {
      const uint32_t num = n_sum[tid];
      sat += num;
      if (kScore) wait_sum += (unsigned long long)num * to_ticks(rec.wait, a.bounds.narrow);
      slot.occ += (int32_t)num;
      slot.q += t_sum[tid];
    }
    if (e0 < R) slot.advance(t_end - t_begin, svc);  // time passes until the next window opens
    t_begin = t_end;
    t_end = t_next;
    // No barrier before the next window's records: everybody has read this window's before the barrier
    // above, and a sum is read and cleared by its own thread.
  }

  if (bad_slot != 0ull) raise_status(a.status, 2u);
  const unsigned long long serves = lane_mask(sat != 0u);
  __syncthreads();  // recs is used again below: .x of entry j = 1 / tbt of a serving instance
  uint32_t sat_w = wave_sum_u32(sat);
  unsigned long long wait_w = wait_sum;
  if (kScore) {
    for (int dlt = 32; dlt >= 1; dlt >>= 1) wait_w += __shfl_xor(wait_w, dlt);
    recs[tid].x = in_mask(serves) ? inv_tbt_first : -1.0f;
  }
  if (lane == 0u) { sat_part[wave] = sat_w; wait_part[wave] = wait_w; }
  __syncthreads();
  if (wave != 0u) return;
  sat_w = 0u;
  wait_w = 0ull;
  for (uint32_t w = 0; w < T / 64u; ++w) { sat_w += sat_part[w]; wait_w += wait_part[w]; }
  float pt = 0.0f;
  if (kScore) {
    // Phi_T: 1 / tbt of the serving instances, added in index order
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const float inv = recs[s * 64 + lane].x;
      for (unsigned long long todo = lane_mask(inv >= 0.0f); todo != 0ull; todo &= todo - 1ull)
        pt = pt + lane_value(inv, (int)__builtin_ctzll(todo));
    }
  }
  if (lane == 0u) write_candidate<kScore>(a, rs, c, sat_w, wait_w, pt);
}

}  // namespace maaso
