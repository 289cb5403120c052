// Instances in the lanes of a wavefront: their live state, its evaluation against the profile, the state
// update between windows, and which of them can be chosen at all.  Shared by the kernels in which a
// wavefront keeps a whole placement in its registers (instance j = s * 64 + lane, S slots per lane).
//
// The arithmetic is device_model.hpp's, operation by operation; what is left out is left out only where
// the result is the same bit for bit (each place says why).
#pragma once

#include "lane_ops.hpp"

#pragma clang fp contract(off)

namespace maaso {

// One instance after profile evaluation, as the triples read it.
struct SlotRecord {
  float a, p, tbt, wait;
  __device__ __forceinline__ SlotRecord of_lane(int l) const {
    return SlotRecord{lane_value(a, l), lane_value(p, l), lane_value(tbt, l), lane_value(wait, l)};
  }
};

// Live state of one instance and what is fixed about it.
struct LiveSlot {
  uint32_t row0;    // its strategy's first table row; row0 + w is the row at effective batch w
  uint32_t B;
  float invB;
  int32_t occ;
  uint64_t q;
  bool configured;  // inside the tables

  // a slot without an instance: empty, inside the tables, never drains
  __device__ __forceinline__ void clear() {
    row0 = 0u; B = 1u; invB = 1.0f; occ = 0; q = 0ull; configured = true;
  }
  __device__ __forceinline__ void load(const ModelParams& mp, uint32_t tp, uint32_t b, int32_t o, uint64_t ticks) {
    configured = tp < mp.n_tp && b != 0u && b <= mp.b_cap;
    row0 = configured ? tp * (mp.b_cap + 1u) : 0u;
    B = b;
    invB = 1.0f / (float)b;
    occ = o;
    q = ticks;
  }

  // stage_instance on the live state, up to the queued prefill: {a, p, tbt}, the expected service time and
  // the wait for a slot past the batch cap.  `tab`: the three tables, entry i of table k at i * kStep + k *
  // stride.  A slot
  // outside the tables gets a record that is never chosen (an infinite wait) and drains with a service
  // time of one second; `bad` has its lane's bit.
  // kPinned: the row is one value ahead of the three loads, so that none of their addresses is worked out from another's.
  template <uint32_t kStep = 1u, bool kPinned = false>
  __device__ __forceinline__ void evaluate(const float* tab, uint32_t stride, const ModelParams& mp, SlotRecord& r,
                                           float& svc, float& past, unsigned long long& bad) const {
    bad = lane_mask(!configured | (occ < 0));
    const uint32_t arriving = (uint32_t)occ + 1u;
    uint32_t w = mp.tbt_mode == 1u ? B : min(arriving, B);
    if (bad != 0ull) w = in_mask(bad) ? 1u : w;
    uint32_t row = kStep == 1u ? row0 + w : (row0 + w) * kStep;
    if (kPinned) asm("" : "+v"(row));
    r.a = tab[row];
    r.p = tab[stride + row];
    r.tbt = tab[2u * stride + row];
    if (mp.pen_kappa != 0.0f) {  // a factor of exactly one without a penalty
      const int32_t over = max(4 * (int32_t)w - 3 * (int32_t)B, 0);  // > 0 iff the batch is > 75 % full
      r.tbt = r.tbt * fmaf(mp.pen_kappa, (float)over * invB, 1.0f);
    }
    svc = mp.s_bar * r.tbt;
    const uint32_t ov = arriving > B ? arriving - B : 0u;  // requests beyond the batch cap
    past = ((float)ov * invB) * svc;
    if (bad != 0ull && in_mask(bad)) {
      r.a = r.p = r.tbt = svc = 1.0f;
      past = INFINITY;
    }
  }

  // The whole wait: queued ticks in seconds on top of `past`.  Ticks below 2^32 (over an hour; `wide`, the
  // same for all lanes, says that some lane has more) convert in one instruction; scaling by 2^-20 is
  // exact, so the fused form rounds once like the sum it stands for.
  __device__ __forceinline__ float wait_with(float past, bool wide) const {
    float qf = (float)(uint32_t)q;
    if (wide) {
      rare_path();
      qf = (float)q;
    }
    return fmaf(qf, 0x1p-20f, past);
  }
  __device__ __forceinline__ bool any_wide() const { return lane_mask((q >> 32) != 0ull) != 0ull; }

  template <bool kPinned = false>
  __device__ __forceinline__ void stage(const float* tab, uint32_t cells, const ModelParams& mp, SlotRecord& r,
                                        float& svc, unsigned long long& bad) const {
    float past;
    evaluate<1u, kPinned>(tab, cells, mp, r, svc, past, bad);
    r.wait = wait_with(past, any_wide());
  }

  // `delta` ticks pass: queued prefill drains, min(occ, B) running requests complete at 1 / svc each.
  __device__ __forceinline__ void advance(uint32_t delta, float svc) {
    q -= (q < (uint64_t)delta) ? q : (uint64_t)delta;
    const float served = (float)min(occ, (int32_t)B) * ((float)delta * 0x1p-20f);
    // 0 <= served < svc: the correctly rounded quotient is below one (at most 1 - 2^-24) and nothing
    // completes - short windows end here
    if (lane_mask(!(served < svc) | (occ < 0)) != 0ull) {
      const float x = served / svc;
      occ -= min(occ, (int32_t)floorf(fminf(x, 2147483520.0f)));
    }
  }
};

// Set of instances, uniform over the wavefront: bit l of m[s] is instance s * 64 + l.
template <int S>
struct InstanceSet {
  unsigned long long m[S];
  __device__ __forceinline__ uint32_t count() const {
    uint32_t n = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) n += (uint32_t)__popcll(m[s]);
    return n;
  }
};

// At most this many instances remove others; past it the rest stays unexamined (the set is then larger
// than need be, never wrong), so that a placement whose instances all differ costs a bounded extra.
constexpr uint32_t kMaxDominators = 16;

// Which instances a request can be admitted to at all, from their records: a set that holds, for every
// request that any instance can serve, the instance the request is given.  Three rules take instances
// out, none of which can take that one (so the order they are applied in does not matter):
//
//  - An instance whose between-token latency is beyond every class, or whose wait and prefill intercept
//    alone are beyond every first-token deadline, is capable of nothing.
//  - Every operation of a triple's slack is monotone under round-to-nearest: the slack never grows when
//    a, p, tbt or wait grows, whatever the request.  With a_k <= a_j, p_k <= p_j, tbt_k <= tbt_j and
//    wait_k <= wait_j, slack_k >= slack_j bit for bit; for k < j ties go to k and j is never chosen.
//  - For k > j the slacks must differ strictly.  They do for every request j is capable of when wait and
//    tbt differ by e_t = 2^-20 max D_ttft and e_b = 2^-20 max D_tbt or more.  With u = 2^-24, the
//    condition evaluated in binary32 leaves true differences of at least e_b - 2u D_tbt = 14u D_tbt and,
//    through the rounded sums, ttft_j - ttft_k >= (16 - 4.1)u D_ttft and e2e_j - e2e_k >= 9.8u D_e2e (a
//    capable j has its latencies below the deadlines, which bounds every rounding).  A margin is
//    (D - x) * (1 / D) with two roundings, so it grows strictly once x falls by more than 4u D.  All
//    three margins of k are then above those of j, and so is the least of them.
//
// Under the shortest-queue rule (kSQ) the last two read: the four comparisons, and k ahead of j in the
// order of (requests on it, index) - k is then capable whenever j is, and before it.  A NaN compares
// false and removes nothing.
//
// Instances that are still in the set when their turn comes remove others, so the number of steps is about
// the number that stay.  That is small, because instances differ in a few strategies and in how loaded
// they are: 3 of 128 mixed instances over windows of 4096 requests (6 without the third rule), 2 of the 64
// of a growth chain over windows of 256.
constexpr float kNarrowSeconds = 512.0f;
struct AdmissionBounds {
  float d_ttft, d_tbt;  // largest deadlines of the classes
  float e_ttft, e_tbt;  // the differences above
  // the largest first-token deadline is below kNarrowSeconds and no wait can come out as no number: the
  // ticks of an admitted request's wait or prefill, and the sum of four prefills, fit 32 bits
  bool narrow;
  // the same, the queue of an instance that admits all of a window stays below 2^32 ticks, and no service time
  // is zero.  NarrowSequence keeps queues in 32 bits on the strength of this alone: an instance admits only while its
  // wait, and so its queue, is within the largest first-token deadline D, and adds at most D per request of the window.
  bool narrow_queue;
};

template <int S, bool kSQ>
__device__ __forceinline__ void find_admissible(const SlotRecord (&rec)[S], const int32_t (&occ)[S], uint32_t n, uint32_t lane,
                                                const AdmissionBounds& lim, InstanceSet<S>& und) {
#pragma unroll
  for (int s = 0; s < S; ++s)
    und.m[s] = lane_mask((uint32_t)s * 64u + lane < n) & lane_mask(rec[s].tbt <= lim.d_tbt) &
               lane_mask(!(rec[s].wait + rec[s].a > lim.d_ttft));
  if (und.count() <= 1u) return;  // nobody to remove
  uint32_t steps = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    for (unsigned long long todo = und.m[s]; todo != 0ull && steps < kMaxDominators; ++steps) {
      const int b = (int)__builtin_ctzll(todo);
      const SlotRecord k = rec[s].of_lane(b);
      const float t_above = k.tbt + lim.e_tbt, w_above = k.wait + lim.e_ttft;
      const int32_t ko = kSQ ? (int32_t)__builtin_amdgcn_readlane(occ[s], b) : 0;
#pragma unroll
      for (int t = 0; t < S; ++t) {
        const unsigned long long ap = lane_mask(k.a <= rec[t].a) & lane_mask(k.p <= rec[t].p);
        const unsigned long long le = ap & lane_mask(k.tbt <= rec[t].tbt) & lane_mask(k.wait <= rec[t].wait);
        // lanes behind instance k in index order
        const unsigned long long behind = t > s ? ~0ull : (t == s ? ~1ull << b : 0ull);
        unsigned long long gone;
        if (kSQ) {
          gone = le & (lane_mask(ko < occ[t]) | (lane_mask(ko == occ[t]) & behind));
        } else {
          gone = (le & behind) | (ap & lane_mask(t_above <= rec[t].tbt) & lane_mask(w_above <= rec[t].wait));
        }
        und.m[t] &= ~gone;
      }
      todo = und.m[s] & (~1ull << b);
    }
  }
}

// The instances a request can be given whether it is admitted or not: only the second rule above, which
// holds for slacks of any sign.  (A blocked request is reported with the largest slack under both
// selection rules.)
template <int S>
__device__ __forceinline__ void find_undominated(const SlotRecord (&rec)[S], uint32_t n, uint32_t lane,
                                                 InstanceSet<S>& und) {
#pragma unroll
  for (int s = 0; s < S; ++s) und.m[s] = lane_mask((uint32_t)s * 64u + lane < n);
  uint32_t steps = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    for (unsigned long long todo = und.m[s]; todo != 0ull && steps < kMaxDominators; ++steps) {
      const int b = (int)__builtin_ctzll(todo);
      const SlotRecord k = rec[s].of_lane(b);
#pragma unroll
      for (int t = s; t < S; ++t) {
        unsigned long long gone = lane_mask(k.a <= rec[t].a) & lane_mask(k.p <= rec[t].p) & lane_mask(k.tbt <= rec[t].tbt) &
                                  lane_mask(k.wait <= rec[t].wait);
        if (t == s) gone &= ~1ull << b;  // those behind it, not itself
        und.m[t] &= ~gone;
      }
      todo = und.m[s] & (~1ull << b);
    }
  }
}

// The first F of a set, in index order: record, index, requests on it (kSQ); entries past its end are
// left as they are.
template <int S, bool kSQ, int F>
__device__ __forceinline__ void first_of(const InstanceSet<S>& set, const SlotRecord (&rec)[S],
                                         const int32_t (&occ)[S], SlotRecord (&fr)[F], uint32_t (&fj)[F],
                                         int32_t (&focc)[F]) {
  InstanceSet<S> left = set;
#pragma unroll
  for (int i = 0; i < F; ++i) {
    bool found = false;
#pragma unroll
    for (int s = 0; s < S; ++s)
      if (!found && left.m[s] != 0ull) {
        const int b = (int)__builtin_ctzll(left.m[s]);
        left.m[s] &= left.m[s] - 1ull;
        fr[i] = rec[s].of_lane(b);
        fj[i] = (uint32_t)(s * 64 + b);
        if (kSQ) focc[i] = (int32_t)__builtin_amdgcn_readlane(occ[s], b);
        found = true;
      }
  }
}

// Shortest-queue rule: a capable instance competes with 512 less its place in the order of (requests on
// it, index) - see queue_rank_value - here among the instances of a set, which is all the order is used
// for.
template <int S>
__device__ __forceinline__ void queue_ranks(const int32_t (&occ)[S], const InstanceSet<S>& und, uint32_t lane,
                                            float (&rank)[S]) {
  uint32_t ahead[S];
#pragma unroll
  for (int s = 0; s < S; ++s) ahead[s] = 0u;
#pragma unroll
  for (int s = 0; s < S; ++s)
    for (unsigned long long todo = und.m[s]; todo != 0ull; todo &= todo - 1ull) {
      const int b = (int)__builtin_ctzll(todo);
      const int32_t ko = (int32_t)__builtin_amdgcn_readlane(occ[s], b);
#pragma unroll
      for (int t = 0; t < S; ++t) {
        const bool before = s < t || (s == t && (uint32_t)b < lane);
        ahead[t] += (ko < occ[t] || (ko == occ[t] && before)) ? 1u : 0u;
      }
    }
#pragma unroll
  for (int s = 0; s < S; ++s) rank[s] = (float)(512u - ahead[s]);
}

}  // namespace maaso
