// Capacity-aware evaluation of candidate deployments over windows of some hundred requests and more, laid out by
// class and prompt length (ordered_windows.hpp): a wavefront per candidate, as sweep_window_kernel with NW = 1, but
// without the block's barriers and without a look at most requests.
//
// What bounds it: vector issue where candidates fill the chip (8192 candidates x 131,072 requests x 128 instances, windows
// of 4096: 1.87 -> 0.67 ms with the batches' prefills added up here, 0.52 with their sums looked up, which a launch of 27 us
// works out for all rows of the tables; 3808 -> 1340 -> 900 vector instructions per wavefront and window);
// the chain of one window after the other where they do not (Alg. 2, 720 deployments x three sets, windows of 256: 1.25 -> 0.70 ms, 3100
// cycles per window of the longest chain: instances 490, search 780, scoring 1530, state 290).  Registers are held to what six or
// seven wavefronts a SIMD take; the first form, which kept the lengths of a window in registers and had a code path per number
// of instances, spilled and was no faster than before.  Batches of 32: 0.58 ms (half as many requests left open, but a pass more).
#pragma once

#include "ordered_windows.hpp"

#pragma clang fp contract(off)

namespace maaso {

struct OrderedSets {
  OrderedSet set[kMaxSweepSets];
  const uint32_t* ticks;  // kTable: batch_ticks_kernel's, of the only set
  uint32_t row_ticks;     // its batches
};

// kSmall: a window is two groups at most.
// (four wavefronts a SIMD with kSmall: held to eight, scalars spill and the chain gets longer.  The scores' forms with two slots a lane
// spill 8 to 12 scalars, the shortest-queue one with the sums 4 vector registers too, those with four slots 16 to 36 scalars.  Held to a wavefront fewer, which spills
// none, the scores took 0.94 to 1.03 times as long, 1.00 on the mean: 1000 to 8192 candidates, 66 to 256 slots, windows of 512 to 4096.)
template <bool kScore, int S, int kLog2, bool kSmall, bool kSQ, bool kTable>
__global__ __launch_bounds__(kAssignThreads, kSmall ? 4 : S == 1 ? 7 : S == 2 ? 6 : 4) void sweep_ordered_kernel(const SweepWindowArgs a,
                                                                                       const OrderedSets o) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* tab = reinterpret_cast<float*>(smem);
  __shared__ ClassRow cls[kMaxSlo];
  constexpr uint32_t kWaves = kAssignThreads / 64;  // candidates of a block

  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  if (tid < a.n_slo) cls[tid] = ClassRow{a.d_ttft[tid], a.d_tbt[tid], a.i_ttft[tid], a.i_tbt[tid]};
  for (uint32_t i = tid; i < 3u * a.cells; i += kAssignThreads) tab[i] = a.tab[i];
  __syncthreads();

  const uint32_t blocks_per_set = (a.n_cand + kWaves - 1u) / kWaves;
  const uint32_t set = blockIdx.x / blocks_per_set;
  const uint32_t c = (blockIdx.x - set * blocks_per_set) * kWaves + wave;
  if (c >= a.n_cand) return;
  const SweepWindowSet rs = resolve_set(a.sets[set]);
  const OrderedSet os = o.set[set];
  const size_t base = (size_t)c * a.i_pad;
  const uint32_t n = min(a.n_inst[c], a.i_pad);

  LiveSlot slot[S];
  unsigned long long bad_slot = 0ull;  // lanes with a slot outside the tables at some window
  uint32_t served[S];
  float inv_tbt_first[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    served[s] = 0u;
    inv_tbt_first[s] = 0.0f;
    slot[s].clear();
    if (j < n)
      slot[s].load(a.mp, a.tp_idx[base + j], a.max_batch[base + j], a.occ[base + j], a.q_ticks[base + j]);
  }
  unsigned long long wait_sum = 0ull;  // queue waits of the requests of this lane's instances, in ticks

  constexpr int kFirst = kSmall ? 2 : 0;
  const Dealt<1, kLog2> deal{0u, lane};
  const uint32_t n_windows = rs.n_req / rs.window + (rs.n_req % rs.window != 0u ? 1u : 0u);
  for (uint32_t w = 0; w < n_windows; ++w) {
    const f32x4 batch = deal.read_batch(os, w, 0u);
    f32x4 len[kFirst ? kFirst : 1];
#pragma unroll
    for (int i = 0; i < kFirst; ++i) len[i] = deal.read_lengths(os, w, 0u, (uint32_t)i);
    const uint32_t gap = os.gap[w];
    SlotRecord rec[S];
    float svc[S];
    int32_t occ[S];  // as the window opens
#pragma unroll
    for (int s = 0; s < S; ++s) {
      occ[s] = slot[s].occ;
      if ((uint32_t)s * 64u >= n && s != 0) continue;  // uniform: no instance in this row of slots
      unsigned long long bad;
      slot[s].stage(tab, a.cells, a.mp, rec[s], svc[s], bad);
      bad_slot |= bad;  // (a lane without an instance is never bad)
      if (kScore && w == 0u) inv_tbt_first[s] = in_mask(bad) ? 0.0f : 1.0f / rec[s].tbt;
    }
    InstanceSet<S> und;
    find_admissible<S, kSQ>(rec, occ, n, lane, a.bounds, und);
    if (und.count() != 0u) {
      uint32_t num[S];  // what this lane's instances take
      unsigned long long ticks[S];
#pragma unroll
      for (int s = 0; s < S; ++s) { num[s] = 0u; ticks[s] = 0ull; }
      auto give = [&](uint32_t j, uint32_t n_j, unsigned long long t_j) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (j == (uint32_t)s * 64u + lane) { num[s] += n_j; ticks[s] += t_j; }
      };
      auto row_of = [&](uint32_t j) __attribute__((always_inline)) {
        uint32_t row = 0;
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (j >> 6 == (uint32_t)s) {
            const uint32_t eff = min(((uint32_t)occ[s] + 1u) | (0u - a.mp.tbt_mode), slot[s].B);
            row = (uint32_t)__builtin_amdgcn_readlane((int)(slot[s].row0 + eff), (int)(j & 63u));
          }
        return row;
      };
      const uint32_t* table = kTable ? o.ticks + (size_t)w * os.batches : nullptr;
      score_window<S, 1, kLog2, kSQ, kFirst, kSmall, kTable>(deal, os, w, batch, len, cls, rec, occ, und, table, o.row_ticks, row_of, give);
#pragma unroll
      for (int s = 0; s < S; ++s) {
        slot[s].occ += (int32_t)num[s];
        slot[s].q += ticks[s];
        served[s] += num[s];
        if (kScore && num[s] != 0u) wait_sum += (unsigned long long)num[s] * to_ticks(rec[s].wait, true);
      }
    }
    if (w + 1u < n_windows) {  // time passes until the next window opens
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (s == 0 || (uint32_t)s * 64u < n) slot[s].advance(gap, svc[s]);
    }
  }

  if (bad_slot != 0ull) raise_status(a.status, 2u);
  uint32_t sat = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) sat += served[s];
  sat = wave_sum_u32(sat);
  float pt = 0.0f;
  if (kScore) {
    for (int d = 32; d >= 1; d >>= 1) wait_sum += __shfl_xor(wait_sum, d);
    // Phi_T: 1 / tbt of the serving instances, added in index order
#pragma unroll
    for (int s = 0; s < S; ++s)
      for (unsigned long long todo = lane_mask(served[s] != 0u); todo != 0ull; todo &= todo - 1ull)
        pt = pt + lane_value(inv_tbt_first[s], (int)__builtin_ctzll(todo));
  }
  if (lane == 0u) write_candidate<kScore>(a, rs, c, sat, wait_sum, pt);
}

}  // namespace maaso
