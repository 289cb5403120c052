// Placer sweep against the state as given: SLO-satisfaction count of every candidate deployment over the
// whole request set (the evaluation of Phi_S(I', R_x) inside Alg. 1; Eq. 3).
//
// A request of class k counts for a candidate iff some instance j meets the between-token deadline and
// wait_j + (a_j + p_j L) meets the first-token one (the end-to-end margin is implied by the two:
// S*tbt + ttft <= S*D_tbt + D_ttft holds in exact arithmetic and a correctly rounded fma is monotone).
// The first-token latency never falls when the prompt length L grows, in binary32 as evaluated, so an
// instance serves exactly the requests of the class up to a longest prompt, a candidate those up to the
// longest of its instances, and the count is a rank among the class's prompt lengths.  The longest
// prompt is found with the latency model itself (a division for a first guess, then evaluations at whole
// lengths until one meets the deadline and its successor does not), so counts are those of evaluating
// every (request, instance) pair, bit for bit, at one threshold per (instance, class) and one look-up
// per (candidate, class).
//
// Launches:
//   1. sweep_hist_kernel, 2. sweep_scatter_kernel - the prompt lengths grouped by (class, bin), 256 bins
//      per class by the leading bits of the binary32 length (eight per octave; two, four ... bins in one
//      where there are many classes and few requests), and the groups' offsets.
//      Beside the second (sweep_prepare_kernel): blocks take groups of candidates, a thread per instance slot
//      evaluates the profile (Eq. 1 row, occupancy penalty, queue wait) and its thresholds, the largest per
//      (candidate, class) meet in LDS.
//   3. sweep_rank_kernel - sixteen lanes per (candidate, class) add the group of the threshold's bin to the
//      lengths below it.  4. sweep_settle_kernel - the best candidate.
// Up to kSmallRequests requests sweep_count_kernel does all of it in one launch: every block groups them in its own
// LDS, and the last block to finish writes the best candidate.  It is also the third launch where the thresholds
// have no room in the workspace, or with some hundred candidates and few requests.
// With few candidates sweep_few_kernel is the only launch: every block compares its share of the requests with all
// thresholds.
//
// What bounds it: the latency of four short launches, each dependent on the one before, and in the second the thresholds.
// 65,536 candidates x 32 slots x 16,384 requests: 457 -> 36.2 -> 33.8 us; 8192 x 128 x 131,072: 5240 -> 38.5 -> 33.8 us;
// 4096 x 32 x 65,536: 127 -> 22.1 -> 21.0 us (every pair evaluated on the vector units; thresholds in the third launch;
// beside the second), the same inputs again and again; with others at every call 37.1 -> 35.0, 40.6 -> 35.8, 22.2 -> 20.0.
// 37 x 13 x 1000: 18 -> 11 us.  The launches by themselves, in a kernel trace with each one's start (which is why they add up
// to more): grouping 3.4 / 5.2 / 3.5, dealing out and thresholds 16.8 / 19.6 / 7.4, ranks 12.0 / 6.6 / 5.8, totals 4.
#pragma once

#include "device_model.hpp"

#pragma clang fp contract(off)

namespace maaso {

constexpr int kSweepThreads = 256;  // 4 wavefronts
constexpr int kWave = 64;
constexpr int kMaxSlo = 16;
constexpr uint32_t kLenBinsLog2 = 8, kLenBins = 1u << kLenBinsLog2;  // per class, or half as many, a quarter ... (LengthGroups)
constexpr uint32_t kSmallRequests = 4096;       // grouped by every block for itself
constexpr uint32_t kMaxGroup = 64;              // candidates a block works on at a time

// Barrier that publishes LDS atomics.  For atomics whose result is unused the compiler emits no wait
// on the LDS counter before the s_barrier of __syncthreads(), and on gfx950 a wavefront reading behind
// that barrier can then see the location without some of the additions (observed as run-to-run
// differences in the per-window admission counts).  Waiting for this wavefront's outstanding LDS
// operations (s_waitcnt lgkmcnt(0), all other counters left at their maxima) before the barrier
// closes that window.  Atomics whose result is used need nothing: the use already waits.
__device__ __forceinline__ void lds_atomics_barrier() {
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __syncthreads();
}

__device__ __forceinline__ void raise_status(uint32_t* status, uint32_t bit) {
  if ((__hip_atomic_load(status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit) == 0u)
    atomicOr(status, bit);
}

// Fill of a few 32-bit words (a kernel, not a memset node, so that a caller may capture the call in a
// HIP graph).
__global__ void fill_u32_kernel(uint32_t* p, uint32_t n, uint32_t v) {
  for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = v;
}

__device__ __forceinline__ float max_no_nan(float x, float y) {
  float r;
  asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}

// A condition as a mask of the wavefront's lanes (scalar register pair), and back.
__device__ __forceinline__ unsigned long long lane_mask(bool p) { return __builtin_amdgcn_ballot_w64(p); }
__device__ __forceinline__ bool in_mask(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Bin of a length >= 0: non-decreasing in it.  Bin 0 is below 1.125, then eight bins per octave.
__device__ __forceinline__ uint32_t length_bin(float L) {
  constexpr uint32_t kFirst = 127u << 3;
  const uint32_t k = __float_as_uint(L) >> 20;
  return k <= kFirst ? 0u : min(k - kFirst, kLenBins - 1u);
}

// Exclusive prefix of the block's per-thread sums, in thread order.  `part`: one word per wavefront.
__device__ __forceinline__ uint32_t block_prefix(uint32_t v, uint32_t* part) {
  const uint32_t lane = threadIdx.x & 63u, wave = threadIdx.x >> 6;
  uint32_t inc = v;
  for (int d = 1; d < 64; d <<= 1) {
    const uint32_t o = __shfl_up(inc, d);
    if (lane >= (uint32_t)d) inc += o;
  }
  if (lane == 63u) part[wave] = inc;
  __syncthreads();
  uint32_t before = inc - v;
  for (uint32_t w = 0; w < wave; ++w) before += part[w];
  return before;
}

// dst[0 .. n) = src[0 .. n), by the block; eight words a thread in flight (one after the other, the 4096
// group totals of sixteen classes were sixteen trips to memory: 10 us of a 15 us launch).
__device__ __forceinline__ void copy_words(uint32_t* dst, const uint32_t* src, uint32_t n) {
  constexpr uint32_t U = 8;
  for (uint32_t i = threadIdx.x; i < n; i += U * kSweepThreads) {
    uint32_t v[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) v[u] = src[min(i + u * kSweepThreads, n - 1u)];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u)
      if (i + u * kSweepThreads < n) dst[i + u * kSweepThreads] = v[u];
  }
}

// Groups of (class, bin): class k's are [k * bins, (k + 1) * bins).
struct LengthGroups {
  uint32_t n_slo;
  uint32_t shift;  // kLenBins >> shift bins per class
  __host__ __device__ __forceinline__ uint32_t bins() const { return kLenBins >> shift; }
  __host__ __device__ __forceinline__ uint32_t count() const { return n_slo * bins(); }
  __device__ __forceinline__ uint32_t of(uint32_t k, float L) const {
    return (k << (kLenBinsLog2 - shift)) + (length_bin(L) >> shift);
  }
  // groups in a row that a thread of a block takes in a pass over all
  __device__ __forceinline__ uint32_t per_thread() const { return (count() + kSweepThreads - 1u) / kSweepThreads; }
};

// kWhole: all kLenBins bins of a class (the usual case, a constant for the compiler).
template <bool kWhole>
__device__ __forceinline__ LengthGroups groups_of(LengthGroups g) {
  if (kWhole) g.shift = 0u;
  return g;
}

struct GroupArgs {
  const uint32_t* prompt_len;
  const uint8_t* slo_class;
  uint32_t n_req;
  LengthGroups groups;
  uint32_t per_block;  // requests per block, contiguous
  uint32_t* hist;      // [groups] zero on entry; the count kernel clears it again
  uint32_t* of_class;  // [n_slo] requests of each class, as hist; or null
  uint32_t* cursor;    // [groups] as hist
  uint32_t* offsets;   // [groups + 1]
  float* sorted;       // [n_req]
  uint32_t* status;
};

// Calls f(group, length) for the requests [r0, r1) of this block whose class exists.
template <bool kFlag, class F>
__device__ __forceinline__ void for_requests(const uint32_t* prompt_len, const uint8_t* slo_class, uint32_t r0,
                                             uint32_t r1, const LengthGroups& groups, uint32_t* status, F f) {
  constexpr uint32_t U = 4;  // loads in flight per thread
  for (uint32_t base = r0; base < r1; base = r1 - base > U * kSweepThreads ? base + U * kSweepThreads : r1) {
    uint32_t k[U];
    float L[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t at = u * kSweepThreads + threadIdx.x;
      const bool in = at < r1 - base;
      k[u] = in ? slo_class[base + at] : 0xffffffffu;
      L[u] = in ? (float)prompt_len[base + at] : 0.0f;
    }
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      if (k[u] < groups.n_slo) f(groups.of(k[u], L[u]), L[u]);
      else if (kFlag && k[u] != 0xffffffffu) raise_status(status, 1u);
    }
  }
}

// LDS words of the two below for n groups.
constexpr uint32_t group_lds_words(uint32_t n) { return n + (n + 15u) / 16u * 17u; }

template <bool kWhole>
__device__ __forceinline__ void count_groups(const GroupArgs& a, uint32_t* h) {
  __shared__ uint32_t of_class[kMaxSlo];
  if (threadIdx.x < kMaxSlo) of_class[threadIdx.x] = 0u;
  const LengthGroups groups = groups_of<kWhole>(a.groups);
  const uint32_t n = groups.count();
  for (uint32_t i = threadIdx.x; i < n; i += kSweepThreads) h[i] = 0u;
  __syncthreads();
  const uint32_t r0 = blockIdx.x * a.per_block;  // the grid covers the requests without overflow
  const uint32_t r1 = a.n_req - r0 > a.per_block ? r0 + a.per_block : a.n_req;
  for_requests<true>(a.prompt_len, a.slo_class, r0, r1, groups, a.status,
                     [&](uint32_t g, float) { atomicAdd(&h[g], 1u); });
  lds_atomics_barrier();
  for (uint32_t i = threadIdx.x; i < n; i += kSweepThreads)
    if (h[i] != 0u) {
      atomicAdd(&a.hist[i], h[i]);
      if (a.of_class) atomicAdd(&of_class[i / groups.bins()], h[i]);
    }
  if (!a.of_class) return;
  lds_atomics_barrier();
  if (threadIdx.x < groups.n_slo && of_class[threadIdx.x] != 0u) atomicAdd(&a.of_class[threadIdx.x], of_class[threadIdx.x]);
}

template <bool kWhole>
__device__ __forceinline__ void deal_out(const GroupArgs& a, uint32_t* h) {
  __shared__ uint32_t part[kSweepThreads / kWave];
  const LengthGroups groups = groups_of<kWhole>(a.groups);
  uint32_t* start = h + groups.count();
  const uint32_t n = groups.count(), per = kWhole ? groups.n_slo : groups.per_thread(), tid = threadIdx.x;
  // where each group starts: every block works it out from the totals, thread t for `per` groups in a row (a
  // word of padding every sixteen keeps the threads' rows off each other's banks)
  auto padded = [](uint32_t i) { return i + (i >> 4); };
  constexpr uint32_t U = 8;  // trips to memory side by side
  for (uint32_t i0 = tid; i0 < n; i0 += U * kSweepThreads) {
    uint32_t v[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) v[u] = a.hist[min(i0 + u * kSweepThreads, n - 1u)];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t i = i0 + u * kSweepThreads;
      if (i < n) { start[padded(i)] = v[u]; h[i] = 0u; }
    }
  }
  __syncthreads();
  uint32_t held[kMaxSlo], sum = 0;
#pragma unroll
  for (uint32_t q = 0; q < kMaxSlo; ++q) {
    const uint32_t i = tid * per + min(q, per - 1u);
    held[q] = start[padded(kWhole ? i : min(i, n - 1u))];
    sum += q < per && (kWhole || i < n) ? held[q] : 0u;
  }
  uint32_t before = block_prefix(sum, part);
#pragma unroll
  for (uint32_t q = 0; q < kMaxSlo; ++q)
    if (q < per && (kWhole || tid * per + q < n)) {
      start[padded(tid * per + q)] = before;
      before += held[q];
    }
  if (blockIdx.x == 0u && tid == kSweepThreads - 1u) a.offsets[n] = before;
  __syncthreads();
  if (blockIdx.x == 0u)
    for (uint32_t i = tid; i < n; i += kSweepThreads) a.offsets[i] = start[padded(i)];
  const uint32_t r0 = blockIdx.x * a.per_block;
  const uint32_t r1 = a.n_req - r0 > a.per_block ? r0 + a.per_block : a.n_req;
  for_requests<false>(a.prompt_len, a.slo_class, r0, r1, groups, a.status,
                      [&](uint32_t g, float) { atomicAdd(&h[g], 1u); });
  lds_atomics_barrier();
  // this block's share of every group it has requests of, eight returning atomics a thread in flight
  for (uint32_t i0 = tid; i0 < n; i0 += U * kSweepThreads) {
    uint32_t own[U], at[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t i = i0 + u * kSweepThreads;
      own[u] = i < n ? h[i] : 0u;
      at[u] = 0u;
      if (own[u] != 0u) at[u] = atomicAdd(&a.cursor[i], own[u]);
    }
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t i = i0 + u * kSweepThreads;
      if (own[u] != 0u) h[i] = start[padded(i)] + at[u];
    }
  }
  __syncthreads();
  for_requests<false>(a.prompt_len, a.slo_class, r0, r1, groups, a.status,
                      [&](uint32_t g, float L) { a.sorted[atomicAdd(&h[g], 1u)] = L; });
}

template <bool kWhole>
__global__ __launch_bounds__(kSweepThreads) void sweep_hist_kernel(const GroupArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  count_groups<kWhole>(a, reinterpret_cast<uint32_t*>(smem));
}

template <bool kWhole>
__global__ __launch_bounds__(kSweepThreads) void sweep_scatter_kernel(const GroupArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  deal_out<kWhole>(a, reinterpret_cast<uint32_t*>(smem));
}

// The longest prompt whose first-token latency meets the deadline, as the bits of its binary32 value plus
// one, or 0 when not even an empty prompt does: from a first guess `n`, the bracket around the answer is
// doubled, then halved (at most some 64 evaluations, whatever the profile).
__device__ __forceinline__ uint32_t search_longest(float a, float p, float wait, float deadline, uint32_t n) {
  auto meets = [&](uint32_t m) { return wait + fmaf(p, (float)m, a) <= deadline; };
  uint32_t lo, hi;  // lo meets the deadline, hi does not
  if (meets(n)) {
    lo = n;
    for (uint32_t step = 1u;; step = step < (1u << 31) ? step << 1 : step) {
      if (lo == 0xffffffffu) return __float_as_uint((float)lo) + 1u;
      hi = lo + min(step, 0xffffffffu - lo);
      if (!meets(hi)) break;
      lo = hi;
    }
  } else {
    hi = n;
    for (uint32_t step = 1u;; step = step < (1u << 31) ? step << 1 : step) {
      if (hi == 0u) return 0u;
      lo = hi > step ? hi - step : 0u;
      if (meets(lo)) break;
      hi = lo;
    }
  }
  while (hi - lo > 1u) {
    const uint32_t mid = lo + ((hi - lo) >> 1);
    if (meets(mid)) lo = mid; else hi = mid;
  }
  return __float_as_uint((float)lo) + 1u;
}

// The same with `inv_p`, about 1 / p: the quotient's whole part is nearly always the answer (it meets the
// deadline, one more does not), and is tried without a branch.  `wanted` false: 0.
__device__ __forceinline__ uint32_t longest_prompt(float a, float p, float wait, float deadline, float inv_p,
                                                   bool wanted) {
  const float guess = fminf(fmaxf(floorf(((deadline - wait) - a) * inv_p), 0.0f), 4294967040.0f);
  const bool now = wait + fmaf(p, guess, a) <= deadline;
  const bool next = wait + fmaf(p, guess + 1.0f, a) <= deadline;
  uint32_t key = now ? __float_as_uint(guess) + 1u : 0u;
  // settled: the quotient, or nothing at all (from 2^24 on guess + 1 may be the guess itself)
  const bool settled = now ? !next : guess == 0.0f;
  if (!settled & wanted) key = search_longest(a, p, wait, deadline, (uint32_t)guess);
  return wanted ? key : 0u;
}

// Accumulators of the count kernel, zero between calls, a cache line each.  Blocks deliver to line
// 1 + (block mod kTotalsLines), the last to deliver to a line hands its totals on to line 0, and the last
// there has them all; whoever is last clears the line.  (Returning atomics on one line take 12 ns each:
// 1024 blocks on a single set of accumulators were 55 us.)
constexpr uint32_t kTotalsLines = 32;
struct alignas(128) SweepTotals {
  unsigned long long best;        // (count << 32) | ~candidate, the largest
  unsigned long long pairs[2];    // (request, instance) pairs past the between-token check: all, without a wait
  uint32_t delivered;             // blocks, or lines
};

// Adds to a line; true, with the line's totals, for the last of `parties`.  Atomics at device scope only,
// each waited for before the delivery is counted: no fence.
__device__ __forceinline__ bool deliver(SweepTotals* t, uint32_t parties, unsigned long long& best,
                                        unsigned long long& pairs, unsigned long long& fresh) {
  const unsigned long long r0 = atomicMax(&t->best, best);
  const unsigned long long r1 = atomicAdd(&t->pairs[0], pairs);
  const unsigned long long r2 = atomicAdd(&t->pairs[1], fresh);
  asm volatile("s_waitcnt vmcnt(0)" : : "v"(r0), "v"(r1), "v"(r2) : "memory");
  if (atomicAdd(&t->delivered, 1u) != parties - 1u) return false;
  best = atomicExch(&t->best, 0ull);
  pairs = atomicExch(&t->pairs[0], 0ull);
  fresh = atomicExch(&t->pairs[1], 0ull);
  atomicExch(&t->delivered, 0u);
  return true;
}

// A block's delivery; true, with the grid's totals, for the last block.  Few blocks meet on line 0 at once.
__device__ __forceinline__ bool deliver_block(SweepTotals* totals, unsigned long long& best,
                                              unsigned long long& pairs, unsigned long long& fresh) {
  if (gridDim.x <= 16u) return deliver(&totals[0], gridDim.x, best, pairs, fresh);
  const uint32_t line = blockIdx.x % kTotalsLines;
  const uint32_t lines = min(gridDim.x, kTotalsLines);
  const uint32_t on_line = (gridDim.x - line + kTotalsLines - 1u) / kTotalsLines;
  return deliver(&totals[1u + line], on_line, best, pairs, fresh) && deliver(&totals[0], lines, best, pairs, fresh);
}

struct CountArgs {
  const float* tab;  // three tables back to back, `cells` entries each
  uint32_t cells;
  ModelParams mp;
  LengthGroups groups;
  float d_ttft[kMaxSlo], d_tbt[kMaxSlo];
  uint32_t n_cand, i_pad;
  const uint32_t* n_inst;
  const uint8_t* tp_idx;
  const uint16_t* max_batch;
  const int32_t* occ;
  const uint64_t* q_ticks;
  uint32_t n_req;
  const uint32_t* prompt_len;  // small form: the requests themselves
  const uint8_t* slo_class;
  const uint32_t* offsets;     // large form: groups and lengths from the two launches before
  const float* sorted;
  uint32_t* clear;             // their histogram and cursors, two words per group, cleared again
  uint32_t group, n_groups;    // candidates per group
  uint32_t* sat_count;
  float* sat_ratio;
  uint32_t* best_cand;
  SweepTotals* totals;             // [1 + kTotalsLines]
  unsigned long long* eval_total;  // [2]
  uint32_t* status;
};

__device__ __forceinline__ uint32_t row_max_u32(uint32_t v) {  // over 16 consecutive lanes
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true));   // quad_perm [1,0,3,2]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true));   // quad_perm [2,3,0,1]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true));  // row_half_mirror
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true));  // row_mirror
  return v;
}
__device__ __forceinline__ uint32_t row_sum_u32(uint32_t v) {
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xb1, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4e, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);
  v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true);
  return v;
}

// kSmall: at most kSmallRequests requests, grouped here.  kRows: i_pad is a multiple of 16, so the 16 lanes
// of a DPP row hold slots of one candidate.
template <bool kSmall, bool kRows, bool kWhole>
__global__ __launch_bounds__(kSweepThreads) void sweep_count_kernel(const CountArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* off = reinterpret_cast<uint32_t*>(smem);                // [groups + 1]
  __shared__ float own[kSmall ? kSmallRequests : 1];                // the grouped lengths
  __shared__ uint32_t longest[kMaxGroup * kMaxSlo];                 // per (candidate, class) of the group
  __shared__ uint32_t cnt[kMaxGroup];
  __shared__ float4 rows[kMaxSlo];                                  // class rows
  __shared__ uint32_t part[kSweepThreads / kWave];
  __shared__ unsigned long long ends[3][kSweepThreads / kWave];

  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const LengthGroups groups = groups_of<kWhole>(a.groups);
  const uint32_t K = groups.n_slo, I = a.i_pad, n = groups.count(), bins = groups.bins();
  if (kSmall) {
    // counts at off[g + 1], then the groups' starts there; dealing the lengths out moves each to its
    // group's end, which is the next group's start
    for (uint32_t i = tid; i <= n; i += kSweepThreads) off[i] = 0u;
    __syncthreads();
    for_requests<true>(a.prompt_len, a.slo_class, 0u, a.n_req, groups, a.status,
                       [&](uint32_t g, float) { atomicAdd(&off[g + 1u], 1u); });
    lds_atomics_barrier();
    const uint32_t per = groups.per_thread(), g0 = min(tid * per, n), g1 = min(g0 + per, n);
    uint32_t sum = 0;
    for (uint32_t g = g0; g < g1; ++g) sum += off[g + 1u];
    uint32_t before = block_prefix(sum, part);
    for (uint32_t g = g0; g < g1; ++g) {
      const uint32_t v = off[g + 1u];
      off[g + 1u] = before;
      before += v;
    }
    __syncthreads();
    for_requests<false>(a.prompt_len, a.slo_class, 0u, a.n_req, groups, a.status,
                        [&](uint32_t g, float L) { own[atomicAdd(&off[g + 1u], 1u)] = L; });
    __syncthreads();
  } else {
    copy_words(off, a.offsets, n + 1u);
    if (blockIdx.x == 0u)
      for (uint32_t i = tid; i < 2u * n; i += kSweepThreads) a.clear[i] = 0u;
    __syncthreads();
  }
  if (tid < K)
    rows[tid] = make_float4(a.d_ttft[tid], a.d_tbt[tid],
                            __uint_as_float(off[(tid + 1u) * bins] - off[tid * bins]), 0.0f);
  auto length_at = [&](uint32_t i) { return kSmall ? own[kSmall ? i : 0u] : a.sorted[i]; };

  unsigned long long best = 0ull;               // of this thread's candidates
  unsigned long long pairs = 0ull, fresh = 0ull;  // of this thread's slots
  for (uint32_t g = blockIdx.x; g < a.n_groups; g = a.n_groups - g > gridDim.x ? g + gridDim.x : a.n_groups) {
    const uint32_t c0 = g * a.group;
    const uint32_t nc = min(a.group, a.n_cand - c0);
    const uint32_t slots = nc * I;
    for (uint32_t i = tid; i < nc * K; i += kSweepThreads) longest[i] = 0u;
    if (tid < nc) cnt[tid] = 0u;
    __syncthreads();
    // two slots a thread at a time, everything read before anything is used
    constexpr uint32_t U = 2;
    for (uint32_t s0 = wave * 64u; s0 < slots; s0 += U * kSweepThreads) {
      uint32_t cl[U], tp[U], B[U], n_inst[U];
      int32_t occ[U];
      uint64_t q[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t s = min(s0 + u * kSweepThreads + lane, slots - 1u);
        cl[u] = s / I;
        const size_t at = (size_t)c0 * I + s;
        n_inst[u] = a.n_inst[c0 + cl[u]];
        tp[u] = a.tp_idx[at]; B[u] = a.max_batch[at]; occ[u] = a.occ[at]; q[u] = a.q_ticks[at];
      }
      Staged st[U];
      float inv_p[U];
      uint32_t reached[U];  // requests whose class the slot's between-token latency suits
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t s = s0 + u * kSweepThreads + lane;
        st[u] = Staged{1.0f, 1.0f, INFINITY, 1.0f, INFINITY};  // absent: suits no class
        if (s < slots && s - cl[u] * I < n_inst[u] &&
            !stage_instance(a.tab, a.cells, a.mp, tp[u], B[u], occ[u], q[u], st[u]))
          raise_status(a.status, 2u);
        inv_p[u] = __builtin_amdgcn_rcpf(st[u].p);
        reached[u] = 0u;
      }
      for (uint32_t k = 0; k < K; ++k) {
        const float4 row = rows[k];  // deadlines, requests of the class
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          const bool in_time = st[u].tbt <= row.y;
          if (lane_mask(in_time) == 0ull) continue;
          reached[u] += in_time ? __float_as_uint(row.z) : 0u;
          uint32_t key = longest_prompt(st[u].a, st[u].p, st[u].wait, row.x, inv_p[u], in_time);
          if (kRows) {
            key = row_max_u32(key);
            if ((lane & 15u) == 0u && key != 0u) atomicMax(&longest[cl[u] * K + k], key);
          } else if (key != 0u) {
            atomicMax(&longest[cl[u] * K + k], key);
          }
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        pairs += reached[u];
        fresh += st[u].wait == 0.0f ? reached[u] : 0u;
      }
    }
    lds_atomics_barrier();
    // the lengths below the threshold's bin, and those of the bin that are not above it: sixteen lanes per
    // (candidate, class), as many more as the block has over (89 candidates x 3 slots, one class, 217k
    // requests, 3000 to a bin: 27 -> 9 us)
    const uint32_t tasks = nc * K;
    const uint32_t width = tasks > 8u ? 4u : tasks > 4u ? 5u : tasks > 2u ? 6u : tasks > 1u ? 7u : 8u;
    static_assert(kSweepThreads == 256, "one (candidate, class) takes at most the block");
    for (uint32_t t = tid >> width; t < tasks; t += kSweepThreads >> width) {
      const uint32_t key = longest[t];
      const uint32_t cl = t / K, k = t - cl * K;
      const uint32_t part_of = tid & ((1u << width) - 1u);
      uint32_t sum = 0;
      if (key != 0u) {
        const float X = __uint_as_float(key - 1u);
        const uint32_t grp = groups.of(k, X);
        const uint32_t b0 = off[grp], b1 = off[grp + 1u];
        constexpr uint32_t U = 8;
        for (uint32_t i = b0 + part_of; i < b1; i = b1 - i > (U << width) ? i + (U << width) : b1) {
          float L[U];
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) {
            L[u] = (u << width) < b1 - i ? length_at(i + (u << width)) : INFINITY;
          }
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) sum += L[u] <= X ? 1u : 0u;
        }
        sum = row_sum_u32(sum) + (part_of == 0u ? b0 - off[k * bins] : 0u);
      }
      if ((lane & 15u) == 0u && sum != 0u) atomicAdd(&cnt[cl], sum);
    }
    lds_atomics_barrier();
    if (tid < nc) {
      const uint32_t c = c0 + tid, v = cnt[tid];
      a.sat_count[c] = v;
      if (a.sat_ratio) a.sat_ratio[c] = a.n_req ? (float)v / (float)a.n_req : 0.0f;
      const unsigned long long kc = ((unsigned long long)v << 32) | (unsigned long long)(~c);
      best = kc > best ? kc : best;
    }
  }
  for (int d = 32; d >= 1; d >>= 1) {
    const unsigned long long o = __shfl_xor(best, d);
    best = o > best ? o : best;
    pairs += __shfl_xor(pairs, d);
    fresh += __shfl_xor(fresh, d);
  }
  if (lane == 0u) { ends[0][wave] = best; ends[1][wave] = pairs; ends[2][wave] = fresh; }
  __syncthreads();
  if (tid == 0u) {
    unsigned long long b = 0ull, e = 0ull, f = 0ull;
    for (int w = 0; w < kSweepThreads / kWave; ++w) {
      b = ends[0][w] > b ? ends[0][w] : b;
      e += ends[1][w];
      f += ends[2][w];
    }
    if (deliver_block(a.totals, b, e, f)) {
      a.eval_total[0] = e;
      a.eval_total[1] = f;
      if (a.best_cand) *a.best_cand = ~(uint32_t)(b & 0xffffffffull);
    }
  }
}

// The large form in four launches: the grouping's two, the second with the thresholds beside it - they need the
// requests of each class, not the groups, and a hundred blocks of 1024 requests leave most of the chip idle for the
// 7 us that dealing the lengths out takes - then the ranks, then a block that settles the totals.  (Delivered by
// atomics from the rank kernel's 2048 blocks, over 32 cache lines, the totals were 5 us and more of its 12 to 17.
// Thresholds beside the first launch as well, 20 / 40 / 60 % of them: 65,536 x 32 slots 36.9 / 35.2 / 35.2 us against 33.6
// with none; tables in LDS and slots read a trip ahead: 8192 x 128 slots 22.7 us for this launch instead of 19.8.)
struct ThresholdArgs {
  const float* tab;
  uint32_t cells;
  ModelParams mp;
  uint32_t n_slo;
  float d_ttft[kMaxSlo], d_tbt[kMaxSlo];
  uint32_t n_cand, i_pad;
  const uint32_t* n_inst;
  const uint8_t* tp_idx;
  const uint16_t* max_batch;
  const int32_t* occ;
  const uint64_t* q_ticks;
  const uint32_t* of_class;    // [n_slo] requests of each class
  uint32_t group, n_groups;    // candidates per group
  uint32_t* longest;           // [n_cand][n_slo] largest longest_prompt of the candidate's slots
  unsigned long long* pairs;   // [blocks][2] (request, instance) pairs past the between-token check: all, without a wait
  uint32_t* status;
};

template <bool kRows>
__device__ __forceinline__ void find_thresholds(const ThresholdArgs& a, uint32_t* longest, uint32_t block, uint32_t blocks) {
  __shared__ float4 rows[kMaxSlo];
  __shared__ unsigned long long ends[2][kSweepThreads / kWave];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t K = a.n_slo, I = a.i_pad;
  if (tid < K) rows[tid] = make_float4(a.d_ttft[tid], a.d_tbt[tid], __uint_as_float(a.of_class[tid]), 0.0f);
  unsigned long long pairs = 0ull, fresh = 0ull;  // of this thread's slots
  for (uint32_t g = block; g < a.n_groups; g = a.n_groups - g > blocks ? g + blocks : a.n_groups) {
    const uint32_t c0 = g * a.group;
    const uint32_t nc = min(a.group, a.n_cand - c0);
    const uint32_t slots = nc * I;
    for (uint32_t i = tid; i < nc * K; i += kSweepThreads) longest[i] = 0u;
    __syncthreads();
    // two slots a thread at a time, everything read before anything is used
    constexpr uint32_t U = 2;
    for (uint32_t s0 = wave * 64u; s0 < slots; s0 += U * kSweepThreads) {
      uint32_t cl[U], tp[U], B[U], n_inst[U];
      int32_t occ[U];
      uint64_t q[U];
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t s = min(s0 + u * kSweepThreads + lane, slots - 1u);
        cl[u] = s / I;
        const size_t at = (size_t)c0 * I + s;
        n_inst[u] = a.n_inst[c0 + cl[u]];
        tp[u] = a.tp_idx[at]; B[u] = a.max_batch[at]; occ[u] = a.occ[at]; q[u] = a.q_ticks[at];
      }
      Staged st[U];
      float inv_p[U];
      uint32_t reached[U];  // requests whose class the slot's between-token latency suits
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        const uint32_t s = s0 + u * kSweepThreads + lane;
        st[u] = Staged{1.0f, 1.0f, INFINITY, 1.0f, INFINITY};  // absent: suits no class
        if (s < slots && s - cl[u] * I < n_inst[u] &&
            !stage_instance(a.tab, a.cells, a.mp, tp[u], B[u], occ[u], q[u], st[u]))
          raise_status(a.status, 2u);
        inv_p[u] = __builtin_amdgcn_rcpf(st[u].p);
        reached[u] = 0u;
      }
      for (uint32_t k = 0; k < K; ++k) {
        const float4 row = rows[k];  // deadlines, requests of the class
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
          const bool in_time = st[u].tbt <= row.y;
          if (lane_mask(in_time) == 0ull) continue;
          reached[u] += in_time ? __float_as_uint(row.z) : 0u;
          uint32_t key = longest_prompt(st[u].a, st[u].p, st[u].wait, row.x, inv_p[u], in_time);
          if (kRows) {
            key = row_max_u32(key);
            if ((lane & 15u) == 0u && key != 0u) atomicMax(&longest[cl[u] * K + k], key);
          } else if (key != 0u) {
            atomicMax(&longest[cl[u] * K + k], key);
          }
        }
      }
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) {
        pairs += reached[u];
        fresh += st[u].wait == 0.0f ? reached[u] : 0u;
      }
    }
    lds_atomics_barrier();
    for (uint32_t i = tid; i < nc * K; i += kSweepThreads) a.longest[(size_t)c0 * K + i] = longest[i];
    __syncthreads();
  }
  for (int d = 32; d >= 1; d >>= 1) {
    pairs += __shfl_xor(pairs, d);
    fresh += __shfl_xor(fresh, d);
  }
  if (lane == 0u) { ends[0][wave] = pairs; ends[1][wave] = fresh; }
  __syncthreads();
  if (tid < 2u) {
    unsigned long long v = 0ull;
    for (int w = 0; w < kSweepThreads / kWave; ++w) v += ends[tid][w];
    a.pairs[2u * block + tid] = v;
  }
}

template <bool kRows, bool kWhole>
__global__ __launch_bounds__(kSweepThreads) void sweep_prepare_kernel(const GroupArgs g, const ThresholdArgs t, uint32_t group_blocks) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* lds = reinterpret_cast<uint32_t*>(smem);
  if (blockIdx.x < group_blocks) deal_out<kWhole>(g, lds);
  else find_thresholds<kRows>(t, lds, blockIdx.x - group_blocks, gridDim.x - group_blocks);
}

struct RankArgs {
  LengthGroups groups;
  uint32_t n_cand, n_req;
  const uint32_t* longest;         // [n_cand][n_slo]
  const uint32_t* offsets;
  const float* sorted;
  uint32_t* clear;                 // histogram and cursors, two words per group, cleared again
  uint32_t* of_class;              // ... and the requests of each class
  uint32_t group, n_groups;        // candidates per group
  uint32_t* sat_count;
  float* sat_ratio;
  unsigned long long* block_best;  // [blocks] (count << 32) | ~candidate, the largest
};

// The lengths below the threshold's bin, and those of the bin that are not above it: 2^width lanes per (candidate,
// class).
template <bool kWhole>
__global__ __launch_bounds__(kSweepThreads) void sweep_rank_kernel(const RankArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* off = reinterpret_cast<uint32_t*>(smem);                // [groups + 1]
  __shared__ uint32_t longest[kMaxGroup * kMaxSlo];
  __shared__ uint32_t cnt[kMaxGroup];
  __shared__ unsigned long long ends[kSweepThreads / kWave];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const LengthGroups groups = groups_of<kWhole>(a.groups);
  const uint32_t K = groups.n_slo, n = groups.count(), bins = groups.bins();
  copy_words(off, a.offsets, n + 1u);
  if (blockIdx.x == 0u) {
    for (uint32_t i = tid; i < 2u * n; i += kSweepThreads) a.clear[i] = 0u;
    if (tid < K) a.of_class[tid] = 0u;
  }
  unsigned long long best = 0ull;
  for (uint32_t g = blockIdx.x; g < a.n_groups; g = a.n_groups - g > gridDim.x ? g + gridDim.x : a.n_groups) {
    const uint32_t c0 = g * a.group;
    const uint32_t nc = min(a.group, a.n_cand - c0);
    const uint32_t tasks = nc * K;
    for (uint32_t i = tid; i < tasks; i += kSweepThreads) longest[i] = a.longest[(size_t)c0 * K + i];
    if (tid < nc) cnt[tid] = 0u;
    __syncthreads();
    const uint32_t width = tasks > 8u ? 4u : tasks > 4u ? 5u : tasks > 2u ? 6u : tasks > 1u ? 7u : 8u;
    const uint32_t part_of = tid & ((1u << width) - 1u), per_pass = kSweepThreads >> width;
    constexpr uint32_t U = 8;  // lengths in flight (two tasks side by side: 34.4 against 34.3 us, four: 37.4)
    for (uint32_t t = tid >> width; t < tasks; t += per_pass) {
      const uint32_t key = longest[t];
      const uint32_t cl = t / K, k = t - cl * K;
      uint32_t sum = 0;
      if (key != 0u) {
        const float X = __uint_as_float(key - 1u);
        const uint32_t grp = groups.of(k, X);
        const uint32_t b0 = off[grp], b1 = off[grp + 1u];
        for (uint32_t i = b0 + part_of; i < b1; i = b1 - i > (U << width) ? i + (U << width) : b1) {
          float L[U];
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) L[u] = (u << width) < b1 - i ? a.sorted[i + (u << width)] : INFINITY;
#pragma unroll
          for (uint32_t u = 0; u < U; ++u) sum += L[u] <= X ? 1u : 0u;
        }
        sum = row_sum_u32(sum) + (part_of == 0u ? b0 - off[k * bins] : 0u);
      }
      if ((lane & 15u) == 0u && sum != 0u) atomicAdd(&cnt[cl], sum);
    }
    lds_atomics_barrier();
    if (tid < nc) {
      const uint32_t c = c0 + tid, v = cnt[tid];
      a.sat_count[c] = v;
      if (a.sat_ratio) a.sat_ratio[c] = a.n_req ? (float)v / (float)a.n_req : 0.0f;
      const unsigned long long kc = ((unsigned long long)v << 32) | (unsigned long long)(~c);
      best = kc > best ? kc : best;
    }
    __syncthreads();
  }
  for (int d = 32; d >= 1; d >>= 1) {
    const unsigned long long o = __shfl_xor(best, d);
    best = o > best ? o : best;
  }
  if (lane == 0u) ends[wave] = best;
  __syncthreads();
  if (tid == 0u) {
    for (int w = 1; w < kSweepThreads / kWave; ++w) best = ends[w] > best ? ends[w] : best;
    a.block_best[blockIdx.x] = best;
  }
}

// The best candidate and the pairs from what the blocks left.  One block.
__global__ __launch_bounds__(1024) void sweep_settle_kernel(const unsigned long long* block_best, uint32_t n_best,
                                                            const unsigned long long* pairs, uint32_t n_pairs,
                                                            uint32_t* best_cand, unsigned long long* eval_total) {
  __shared__ unsigned long long ends[3][1024 / kWave];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  unsigned long long best = 0ull, all = 0ull, fresh = 0ull;
#pragma unroll 4
  for (uint32_t i = tid; i < n_best; i += 1024u) best = block_best[i] > best ? block_best[i] : best;
#pragma unroll 4
  for (uint32_t i = tid; i < n_pairs; i += 1024u) { all += pairs[2u * i]; fresh += pairs[2u * i + 1u]; }
  for (int d = 32; d >= 1; d >>= 1) {
    const unsigned long long o = __shfl_xor(best, d);
    best = o > best ? o : best;
    all += __shfl_xor(all, d);
    fresh += __shfl_xor(fresh, d);
  }
  if (lane == 0u) { ends[0][wave] = best; ends[1][wave] = all; ends[2][wave] = fresh; }
  __syncthreads();
  if (tid == 0u) {
    for (int w = 1; w < 1024 / kWave; ++w) {
      best = ends[0][w] > best ? ends[0][w] : best;
      all += ends[1][w];
      fresh += ends[2][w];
    }
    eval_total[0] = all;
    eval_total[1] = fresh;
    if (best_cand) *best_cand = ~(uint32_t)(best & 0xffffffffull);
  }
}

// The same counts in one launch where there are few candidates: every block works out the thresholds of all of
// them and compares its share of the requests with each, a count per candidate from the lanes' masks.  Grouping the lengths costs two launches and pays only where a length is looked up often.
constexpr uint32_t kFewCandidates = 128;
__global__ __launch_bounds__(kSweepThreads) void sweep_few_kernel(const CountArgs a) {
  __shared__ uint32_t longest[kMaxSlo * (kFewCandidates + 1u)];  // [class][candidate], rows of odd length
  __shared__ uint32_t cnt[kFewCandidates];
  __shared__ uint32_t suits[2][kMaxSlo], of_class[kMaxSlo];  // slots a class can use (all; without a wait); requests
  __shared__ unsigned long long ends[kSweepThreads / kWave];
  __shared__ uint32_t last;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, wave = tid >> 6;
  const uint32_t K = a.groups.n_slo, I = a.i_pad, C = a.n_cand, slots = C * I, pitch = C | 1u;
  constexpr uint32_t U = 4;
  const uint32_t per_trip = gridDim.x * U * kSweepThreads;  // the host keeps it far below 2^32
  // this block's first requests are on their way while the thresholds are worked out
  uint32_t r0 = blockIdx.x * U * kSweepThreads;
  uint32_t k[U], key[U];
  auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const uint32_t at = u * kSweepThreads + tid;
      const bool in = r0 < a.n_req && at < a.n_req - r0;
      k[u] = in ? a.slo_class[r0 + at] : 0xffffffffu;
      key[u] = in ? a.prompt_len[r0 + at] : 0u;
    }
  };
  fetch();
  for (uint32_t i = tid; i < K * pitch; i += kSweepThreads) longest[i] = 0u;
  if (tid < C) cnt[tid] = 0u;
  if (tid < K) { suits[0][tid] = 0u; suits[1][tid] = 0u; of_class[tid] = 0u; }
  __syncthreads();
  for (uint32_t s0 = wave * 64u; s0 < slots; s0 += kSweepThreads) {
    const uint32_t s = min(s0 + lane, slots - 1u), c = s / I;
    Staged st{1.0f, 1.0f, INFINITY, 1.0f, INFINITY};  // absent: suits no class
    if (s0 + lane < slots && s - c * I < a.n_inst[c] &&
        !stage_instance(a.tab, a.cells, a.mp, a.tp_idx[s], a.max_batch[s], a.occ[s], a.q_ticks[s], st))
      raise_status(a.status, 2u);
    const float inv_p = __builtin_amdgcn_rcpf(st.p);
    for (uint32_t q = 0; q < K; ++q) {
      const bool in_time = st.tbt <= a.d_tbt[q];
      const unsigned long long m = lane_mask(in_time);
      if (m == 0ull) continue;
      const unsigned long long f = lane_mask(in_time && st.wait == 0.0f);
      if (lane == 0u) {
        atomicAdd(&suits[0][q], (uint32_t)__popcll(m));
        atomicAdd(&suits[1][q], (uint32_t)__popcll(f));
      }
      const uint32_t x = longest_prompt(st.a, st.p, st.wait, a.d_ttft[q], inv_p, in_time);
      if (x != 0u) atomicMax(&longest[q * pitch + c], x);
    }
  }
  lds_atomics_barrier();
  uint32_t mine[2] = {0u, 0u};
  while (r0 < a.n_req) {  // the same for all threads of the block
    uint32_t have[U], row[U];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) {
      const bool ok = k[u] < K;
      if (!ok && k[u] != 0xffffffffu) raise_status(a.status, 1u);
      // thresholds are the bits of a length plus one: a request counts when its own bits are below
      have[u] = ok ? __float_as_uint((float)key[u]) : 0xffffffffu;
      row[u] = (ok ? k[u] : 0u) * pitch;
    }
    for (uint32_t q = 0; q < K; ++q) {
      uint32_t sum = 0;
#pragma unroll
      for (uint32_t u = 0; u < U; ++u) sum += (uint32_t)__popcll(lane_mask(k[u] == q));
      if (lane == 0u) atomicAdd(&of_class[q], sum);
    }
    r0 = a.n_req - r0 > per_trip ? r0 + per_trip : a.n_req;
    fetch();
    // candidate c's count in lane c mod 64; four candidates' thresholds read ahead of their use
    constexpr uint32_t V = 4;
    for (uint32_t c0 = 0; c0 < C; c0 += V) {
      uint32_t x[V][U];
#pragma unroll
      for (uint32_t v = 0; v < V; ++v)
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) x[v][u] = longest[row[u] + min(c0 + v, C - 1u)];
#pragma unroll
      for (uint32_t v = 0; v < V; ++v) {
        uint32_t sum = 0;
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) sum += (uint32_t)__popcll(lane_mask(have[u] < x[v][u]));
        const uint32_t c = c0 + v;
        if (c < 64u) mine[0] += lane == c ? sum : 0u;
        else mine[1] += lane == c - 64u ? sum : 0u;  // (c >= C: nobody's)
      }
    }
  }
#pragma unroll
  for (uint32_t w = 0; w < 2u; ++w) {
    const uint32_t c = w * 64u + lane;
    if (c < C && mine[w] != 0u) atomicAdd(&cnt[c], mine[w]);
  }
  lds_atomics_barrier();
  if (tid < C) {
    const uint32_t before = atomicAdd(&a.clear[tid], cnt[tid]);  // zero between calls
    asm volatile("s_waitcnt vmcnt(0)" : : "v"(before) : "memory");
  }
  __syncthreads();
  if (tid == 0u) {
    unsigned long long b = 0ull, e = 0ull, f = 0ull;
    for (uint32_t q = 0; q < K; ++q) {
      e += (unsigned long long)suits[0][q] * of_class[q];
      f += (unsigned long long)suits[1][q] * of_class[q];
    }
    const bool all = deliver_block(a.totals, b, e, f);
    last = all ? 1u : 0u;
    if (all) { a.eval_total[0] = e; a.eval_total[1] = f; }
  }
  __syncthreads();
  if (last == 0u) return;
  unsigned long long best = 0ull;
  if (tid < C) {
    const uint32_t v = atomicExch(&a.clear[tid], 0u);
    a.sat_count[tid] = v;
    if (a.sat_ratio) a.sat_ratio[tid] = a.n_req ? (float)v / (float)a.n_req : 0.0f;
    best = ((unsigned long long)v << 32) | (unsigned long long)(~tid);
  }
  for (int d = 32; d >= 1; d >>= 1) {
    const unsigned long long o = __shfl_xor(best, d);
    best = o > best ? o : best;
  }
  if (lane == 0u) ends[wave] = best;
  __syncthreads();
  if (tid == 0u && a.best_cand) {
    for (int w = 1; w < kSweepThreads / kWave; ++w) best = ends[w] > best ? ends[w] : best;
    *a.best_cand = ~(uint32_t)(best & 0xffffffffull);
  }
}

// ---------------------------------------------------------------------------------------------
// Of a windowed sweep's counts: ratio[c] = count[c] / R and the best candidate - largest count, lowest
// index on ties (Alg. 1 keeps the best-scoring deployment).  One block, so its duration is the number of
// dependent trips to memory: eight elements per thread are requested before any is used.
__global__ __launch_bounds__(1024) void sweep_finalize_kernel(const uint32_t* __restrict__ sat_count,
                                                              uint32_t n_cand, uint32_t n_req,
                                                              float* __restrict__ sat_ratio,
                                                              uint32_t* __restrict__ best_cand) {
  __shared__ unsigned long long best[16];
  constexpr uint32_t kBatch = 8;
  const uint32_t stride = kBatch * blockDim.x;
  const float fr = (float)n_req;
  unsigned long long key = 0ull;  // (count << 32) | ~index: max key = max count, then min index
  for (uint32_t c0 = threadIdx.x; c0 < n_cand; c0 = n_cand - c0 > stride ? c0 + stride : n_cand) {
    uint32_t n[kBatch];
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u) {
      const uint32_t at = u * blockDim.x;
      n[u] = at < n_cand - c0 ? sat_count[c0 + at] : 0u;
    }
#pragma unroll
    for (uint32_t u = 0; u < kBatch; ++u) {
      const uint32_t at = u * blockDim.x;
      if (at >= n_cand - c0) continue;
      const uint32_t c = c0 + at;
      if (sat_ratio) sat_ratio[c] = n_req ? (float)n[u] / fr : 0.0f;
      const unsigned long long kc = ((unsigned long long)n[u] << 32) | (unsigned long long)(~c);
      key = kc > key ? kc : key;
    }
  }
  for (int d = 32; d >= 1; d >>= 1) {
    const unsigned long long o = __shfl_xor(key, d);
    key = o > key ? o : key;
  }
  if ((threadIdx.x & 63u) == 0u) best[threadIdx.x >> 6] = key;
  __syncthreads();
  if (threadIdx.x == 0 && best_cand) {
    for (uint32_t w = 1; w < (blockDim.x >> 6); ++w) key = best[w] > key ? best[w] : key;
    *best_cand = ~(uint32_t)(key & 0xffffffffull);
  }
}

}  // namespace maaso
