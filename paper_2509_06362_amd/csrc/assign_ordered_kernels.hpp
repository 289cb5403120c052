// Distributor over an online request stream in windows of some hundred requests and more, in two launches beside the one
// that lays the requests out (ordered_windows.hpp): one block takes the placement's state through the windows,
// for which it needs what every instance was given but not by which request, and leaves the records that each window's
// requests met; then all requests are scored against their window's records at once.
//
// Nothing is exchanged between blocks, and a window in which no instance can admit anything - most of them once a
// placement is overloaded - costs no look at its requests.
//
// 64 instances, 1024 windows of 4096 requests, of which 188 admit something: 2.75 ms in the persistent kernel -> 0.58 (26 us to lay
// out, 27 us to score all requests, the rest the states).  What bounds the states: the chain of windows on one wavefront a SIMD, some
// 0.25 us for a window that admits nothing, 1.5 for the others - instances, search, bounds, sums, one barrier - and
// trips to memory of over a microsecond where a window is not expected to admit.  The states' forms of two and four slots a lane keep 19 to 69 scalars in
// lanes of vector registers; none spills to memory.
#pragma once

#include <type_traits>

#include "assign_kernels.hpp"
#include "ordered_windows.hpp"

#pragma clang fp contract(off)

namespace maaso {

// Windows w0 .. w0 + n_windows - 1 of a stream, and where their records go: window w's n_pad from w * n_pad on.
struct StateRun {
  uint32_t n_req, window, w0, n_windows;
  float4* recs;   // {a, p, tbt, wait}
  int32_t* occ;   // requests on the instances (shortest-queue rule only)
};

// NW wavefronts share a window's requests; each keeps the whole state and advances it by itself.  One more writes the
// records: a wavefront's loads would wait for its stores.
template <int S, int NW, bool kSQ>
__global__ __launch_bounds__((NW + 1) * 64) void assign_states_kernel(const AssignArgs a, const OrderedSet os, const StateRun run) {
  constexpr uint32_t T = (NW + 1) * 64;
  static_assert(T >= 64u * S, "a thread per sum");
  extern __shared__ __align__(16) unsigned char smem[];
  float* tab = reinterpret_cast<float*>(smem);
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ uint32_t n_sum[kSumBuffers][64 * S];  // what a window's requests add (see kSumBuffers)
  __shared__ unsigned long long t_sum[kSumBuffers][64 * S];

  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const bool scores = wave < (uint32_t)NW;
  if (tid < a.n_slo) cls[tid] = ClassRow{a.d_ttft[tid], a.d_tbt[tid], a.i_ttft[tid], a.i_tbt[tid]};
  for (uint32_t i = tid; i < 3u * a.cells; i += T) tab[i] = a.tab[i];
  for (uint32_t i = tid; i < kSumBuffers * 64u * S; i += T) { (&n_sum[0][0])[i] = 0u; (&t_sum[0][0])[i] = 0ull; }
  const PlacementRow row = select_row(a);
  const uint32_t n = (uint32_t)__builtin_amdgcn_readfirstlane((int)row.n);
  LiveSlot slot[S];
  uint32_t served = 0;
  unsigned long long bad_slot = 0ull;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    slot[s].clear();
    if (j < n) slot[s].load(a.mp, row.tp_idx[j], row.max_batch[j], row.occ[j], row.q_ticks[j]);
  }
  __syncthreads();

  constexpr int kLog2 = 6, kFirst = 5;  // five groups each: windows of up to 4096 requests
  const Dealt<NW, kLog2> deal{scores ? wave : 0u, lane};
  const uint32_t last = (uint32_t)(((uint64_t)run.n_req + run.window - 1u) / run.window) - 1u - run.w0;  // behind it no time passes
  const uint32_t end = run.n_windows;
  auto read_gaps = [&](uint32_t w) __attribute__((always_inline)) { return w + lane < end ? os.gap[w + lane] : 0u; };
  uint32_t gaps = read_gaps(0u), gaps_next = read_gaps(64u);
  asm volatile("" : "+v"(gaps));
  uint32_t buf = 0;
  SlotRecord rec[S];
  float svc[S];
  uint32_t at_w[S];  // effective batch that rec and svc were evaluated at; 0: at none
#pragma unroll
  for (int s = 0; s < S; ++s) at_w[s] = 0u;
  // The windows, for a wavefront that scores and for the one that writes: each waits for its own memory operations only.
  auto walk = [&](auto scores_) __attribute__((always_inline)) {
    constexpr bool kScores = decltype(scores_)::value;
    uint32_t w = 0, gap = 0;
    int32_t occ[S];
    // Evaluates the instances for window w; whether one may admit something in it or the window behind it (a wait
    // shortens by some two gaps a window).
    auto open = [&]() __attribute__((always_inline)) {
      if ((w & 63u) == 0u && w != 0u) {
        asm volatile("" : "+v"(gaps_next));  // arrived here: no other window waits for memory on its account
        gaps = gaps_next;
        gaps_next = read_gaps(w + 64u);
      }
      gap = (uint32_t)__builtin_amdgcn_readlane((int)gaps, (int)(w & 63u));
      const float reach = fmaf(3.0f, (float)gap * 0x1p-20f, a.bounds.d_ttft);
      unsigned long long near = 0ull;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        occ[s] = slot[s].occ;
        if ((uint32_t)s * 64u >= n && s != 0) continue;  // uniform: no instance in this row of slots
        // the table rows only where an effective batch changed: a full instance's stays what it is
        const uint32_t arriving = (uint32_t)slot[s].occ + 1u;
        const uint32_t eff = min(arriving | (0u - a.mp.tbt_mode), slot[s].B);
        float past = ((float)__builtin_elementwise_sub_sat(arriving, slot[s].B) * slot[s].invB) * svc[s];
        if ((lane_mask(eff != at_w[s]) | lane_mask(!slot[s].configured) | lane_mask(slot[s].occ < 0)) != 0ull) {
          unsigned long long bad;
          slot[s].evaluate(tab, a.cells, a.mp, rec[s], svc[s], past, bad);
          bad_slot |= bad;
          at_w[s] = in_mask(bad) ? 0u : eff;  // a record that stands in for none is not kept (an occupancy may return from below zero)
        }
        rec[s].wait = slot[s].wait_with(past, slot[s].any_wide());
        near |= lane_mask(!(rec[s].wait > reach)) & lane_mask((uint32_t)s * 64u + lane < n);
      }
      return near != 0ull;
    };
    auto record = [&]() __attribute__((always_inline)) {
      if (kScores) return;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const uint32_t j = (uint32_t)s * 64u + lane;
        if (j >= n) continue;
        run.recs[(size_t)w * a.i_pad + j] = make_float4(rec[s].a, rec[s].p, rec[s].tbt, rec[s].wait);
        if (kSQ) run.occ[(size_t)w * a.i_pad + j] = occ[s];
      }
    };
    auto ask = [&](uint32_t of, f32x4& batch, f32x4 (&len)[kFirst]) __attribute__((always_inline)) {
      batch = deal.read_batch(os, of, 0u);
#pragma unroll
      for (int i = 0; i < kFirst; ++i) len[i] = deal.read_lengths(os, of, 0u, (uint32_t)i);
    };
    // time passes until the next window opens; false behind the last one of this launch
    auto advance = [&]() __attribute__((always_inline)) {
      if (w != last) {
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (s == 0 || (uint32_t)s * 64u < n) slot[s].advance(gap, svc[s]);
      }
      return ++w != end;
    };

    bool near = open();
    for (;;) {
      while (!near) {  // nobody can admit anything
        record();
        if (!advance()) return;
        near = open();
      }
      f32x4 batch{}, len[kFirst] = {};
      if (kScores) ask(w, batch, len);
      for (;;) {
        record();
        InstanceSet<S> und;
        find_admissible<S, kSQ>(rec, occ, n, lane, a.bounds, und);
        if (kScores) {
          arrived(batch);
#pragma unroll
          for (int i = 0; i < kFirst; ++i) arrived(len[i]);
        }
        f32x4 next_batch{}, next_len[kFirst] = {};
        if (kScores) ask(min(w + 1u, end - 1u), next_batch, next_len);
        if (und.count() != 0u) {  // (the same in every wavefront)
          if (kScores) {
            auto give = [&](uint32_t j, uint32_t n_j, unsigned long long t_j) __attribute__((always_inline)) {
              if (lane == 0u) {
                atomicAdd(&n_sum[buf][j], n_j);
                atomicAdd(&t_sum[buf][j], t_j);
              }
            };
            score_window<S, NW, kLog2, kSQ, kFirst, false, false>(deal, os, w, batch, len, cls, rec, occ, und, nullptr, 0u,
                                                                  [](uint32_t) { return 0u; }, give);
          }
          const uint32_t free = cleared_sum_buffer(buf);  // clean before anyone passes this barrier
          if (tid < 64u * S) { n_sum[free][tid] = 0u; t_sum[free][tid] = 0ull; }
          lds_atomics_barrier();
#pragma unroll
          for (int s = 0; s < S; ++s) {
            const uint32_t num = n_sum[buf][s * 64 + lane];
            slot[s].occ += (int32_t)num;
            slot[s].q += t_sum[buf][s * 64 + lane];
            served += num;
          }
          buf = next_sum_buffer(buf);
        }
        if (!advance()) return;
        near = open();
        if (!near) break;
        batch = next_batch;
#pragma unroll
        for (int i = 0; i < kFirst; ++i) len[i] = next_len[i];
      }
    }
  };
  if (scores) walk(std::true_type{});
  else walk(std::false_type{});

  if (bad_slot != 0ull) raise_status(a.status, 2u);
  if (wave != 0u) return;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    if (j < n) { row.occ[j] = slot[s].occ; row.q_ticks[j] = slot[s].q; }
  }
  for (int d = 32; d >= 1; d >>= 1) served += __shfl_xor(served, d);
  if (lane == 0u && a.n_satisfied) *a.n_satisfied = (run.w0 == 0u ? 0ull : *a.n_satisfied) + served;
}

// A block's requests, per_block at most of one window, against the window's records: as assign_static_kernel.
template <bool kLat, int V, bool kSQ, int LIST>
__global__ __launch_bounds__(kAssignThreads) void assign_recorded_kernel(const AssignArgs a, const StateRun run,
                                                                         uint32_t blocks_per_window, uint32_t per_block) {
  constexpr bool kAll = LIST == 0;
  constexpr int kList = LIST ? 256 + 3 : 1;
  static_assert(!kAll || !kSQ, "ranks come with a list");
  __shared__ float4 recs[256 + 3];  // whole trips of four are read
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ float4 adm_recs[kList], rep_recs[kList];
  __shared__ uint32_t adm_idx[kList], rep_idx[kList], sizes[2];
  __shared__ float adm_rank[kSQ ? kList : 1];
  __shared__ int32_t occ_s[kSQ ? 256 : 1];
  const uint32_t w = blockIdx.x / blocks_per_window, part = blockIdx.x - w * blocks_per_window;
  const uint64_t s0 = (uint64_t)(run.w0 + w) * run.window;
  const uint64_t e0 = min(s0 + run.window, (uint64_t)run.n_req);
  const uint64_t r0 = s0 + (uint64_t)part * per_block, r1 = min(r0 + per_block, e0);
  if (r0 >= r1) return;  // the last window may be short
  const uint64_t g0 = r0 / V + threadIdx.x, g1 = r0 / V + (r1 - r0) / V;  // groups of V requests (V = 4: r0 is a multiple)
  RequestVec cur{}, nxt{};
  if (V == 4 && g0 < g1) cur = load_request_vec(a, g0 * V);
  const uint32_t n = select_row(a).n;
  for (uint32_t j = threadIdx.x; j < n; j += kAssignThreads) {
    recs[j] = run.recs[(size_t)w * a.i_pad + j];
    if (kSQ) occ_s[j] = run.occ[(size_t)w * a.i_pad + j];
  }
  if (threadIdx.x < a.n_slo) {
    const uint32_t k = threadIdx.x;
    cls[k] = ClassRow{a.d_ttft[k], a.d_tbt[k], a.i_ttft[k], a.i_tbt[k]};
  }
  __syncthreads();
  if (!kAll) {
    if (threadIdx.x < 64u)  // the two lists side by side, a wavefront each
      list_candidates<LIST ? LIST : 1, kSQ, false>(a.bounds, recs, occ_s, n, threadIdx.x, adm_recs, adm_idx, adm_rank, &sizes[0]);
    else if (threadIdx.x < 128u)
      list_candidates<LIST ? LIST : 1, kSQ, true>(a.bounds, recs, occ_s, n, threadIdx.x - 64u, rep_recs, rep_idx, nullptr, &sizes[1]);
    __syncthreads();
  }
  const CandidateList adm{kAll ? recs : adm_recs, kAll ? nullptr : adm_idx, adm_rank,
                          kAll ? n : (uint32_t)__builtin_amdgcn_readfirstlane((int)sizes[0])};
  const CandidateList rep{rep_recs, rep_idx, nullptr, LIST ? (uint32_t)__builtin_amdgcn_readfirstlane((int)sizes[1]) : 0u};
  for (uint64_t g = g0; g < g1; g += kAssignThreads) {
    if (V == 4 && g + kAssignThreads < g1) nxt = load_request_vec(a, (g + kAssignThreads) * V);
    assign_requests<kLat, V, 0, kSQ, kAll>(a, g * V, n, recs, cls, adm, rep, nullptr, nullptr, V == 4 ? &cur : nullptr);
    cur = nxt;
  }
  if (V > 1) {  // the ragged tail, one request per thread
    const uint64_t r = g1 * V + threadIdx.x;
    if (r < r1) assign_requests<kLat, 1, 0, kSQ, kAll>(a, r, n, recs, cls, adm, rep, nullptr, nullptr);
  }
}

}  // namespace maaso
