// Placer with capacity-aware scoring: every candidate deployment is run through the windowed
// distributor on its own copy of its instance state - the stand-in for the paper's virtual-slot
// simulator (Sec. V-A "Simulator Implementation") inside the evaluation of a candidate (Alg. 1).
//
// Candidates do not interact, so a wavefront (or, where there are few candidates, a block of four) owns one
// and walks the windows by itself: no device-wide barrier.  Its lanes hold the instances (state, profile
// evaluation, the drain between windows); per window it works out which instances a request can be
// admitted to at all (find_admissible: 1 to 4 in nineteen windows of twenty) and scores the requests,
// lanes = requests, against those alone.  (Few candidates and windows of up to a few hundred requests have a
// form of their own, sweep_block_kernels.hpp, and windows of a few requests another, sweep_seq_kernels.hpp.)
//
// What a window's admitted requests add up to is kept in registers where a few instances are left, and in
// LDS where more are: an addition per request unless a whole wavefront chose one instance, then every lane
// fetches its instances' sums (a trip per instance chosen before: 1024 candidates x 128 jittered slots,
// windows of 256: 11.7 -> 9.4 us a window; every instance scored: 10.8).
//
// What bounds it: vector issue at windows of thousands (8192 candidates x 131,072 requests x 128
// instances, windows of 4096: 26.8 ms with every instance scored, 1.83 ms here; 238 vector and 90 scalar
// instructions per wavefront and 256 requests), the chain of one window after the other at short ones
// (Alg. 2, 720 deployments x three sets, windows of 256: 2.6 -> 1.24 ms, 2.4 us per window of the longest
// chain; 214 vector and 155 scalar instructions per window).  Both of these now go to sweep_ordered_kernels.hpp; this kernel
// keeps the shapes on the other side of sweep_lays_out, deadlines of 512 s and more, and captured launches.
#pragma once

#include "assign_kernels.hpp"
#include "live_slots.hpp"
#include "window_rules.hpp"

#pragma clang fp contract(off)

namespace maaso {

// One request set and the outputs of scoring every candidate against it.
struct SweepWindowSet {
  uint32_t n_req;
  uint32_t window;  // requests per window (>= 1)
  const uint32_t* prompt_len;
  const uint32_t* out_len;
  const uint8_t* slo_class;
  const uint32_t* arrival_ticks;
  uint32_t* sat_count;
  // composite serving score (kScore kernels only); every output may be null
  float* phi_s;
  float* phi_t;
  float* phi_l;
  float* score;
  // One side of a split whose position only the device knows (Alg. 2 scores R_t and R_l straight
  // after the split, without the host reading |R_t| back): with split_at set, the pointers above
  // address the whole split array of n_req requests and the set is its first *split_at requests
  // (side == 1) or the rest (side == 2).
  const uint32_t* split_at;
  uint32_t side;
};

constexpr int kMaxSweepSets = 4;

// The set a block works on, with a device-side split applied.
__device__ __forceinline__ SweepWindowSet resolve_set(const SweepWindowSet& in) {
  SweepWindowSet rs = in;
  if (in.split_at) {
    const uint32_t at = min(*in.split_at, in.n_req);
    const uint32_t off = in.side == 1u ? 0u : at;
    rs.n_req = in.side == 1u ? at : in.n_req - at;
    rs.prompt_len += off;
    rs.out_len += off;
    rs.slo_class += off;
    if (rs.arrival_ticks) rs.arrival_ticks += off;
  }
  return rs;
}

struct SweepWindowArgs {
  const float* tab;
  uint32_t cells;
  ModelParams mp;
  uint32_t n_slo;
  float d_ttft[kMaxSlo], d_tbt[kMaxSlo], i_ttft[kMaxSlo], i_tbt[kMaxSlo];
  AdmissionBounds bounds;
  uint32_t n_cand, i_pad;
  const uint32_t* n_inst;
  const uint8_t* tp_idx;
  const uint16_t* max_batch;
  const int32_t* occ;
  const uint64_t* q_ticks;
  // Block b scores candidate b % n_cand against set b / n_cand: the sets are independent runs over
  // the same candidates (Alg. 2 scores every deployment against R_t, R_l and all of R), listed
  // longest first so that the blocks that run longest start first.
  uint32_t n_sets;
  SweepWindowSet sets[kMaxSweepSets];
  uint32_t* status;
  float alpha, beta, gamma_t, gamma_l;
};

// A request as it comes from memory, and with everything that depends on the request alone worked out
// (its class row, the end-to-end deadline and its reciprocal).
constexpr uint32_t kNoRequest = 0x80000000u;  // in place of the class where there is no request
struct RequestRaw {
  uint32_t pl, ol, k;
};
struct RequestSide {
  float4 u;  // prompt length, first-token deadline, between-token deadline, output length
  float4 w;  // reciprocals of the two deadlines, end-to-end deadline, its reciprocal
};

// Request r0 + i, if that is before `end`.
__device__ __forceinline__ RequestRaw fetch_request(const SweepWindowSet& rs, uint32_t r0, uint32_t i, uint32_t end) {
  RequestRaw raw{0u, 0u, kNoRequest};
  const uint32_t r = r0 + i;
  if (r0 < end && i < end - r0) { raw.pl = rs.prompt_len[r]; raw.ol = rs.out_len[r]; raw.k = rs.slo_class[r]; }
  return raw;
}

// No request, or a class out of range: deadlines that no latency meets.
__device__ __forceinline__ RequestSide request_side(const RequestRaw& raw, uint32_t n_slo, const ClassRow* cls,
                                                    uint32_t* status) {
  const bool live = raw.k < n_slo;
  if (!live && raw.k != kNoRequest) raise_status(status, 1u);
  const ClassRow cr = cls[live ? raw.k : 0u];
  const float L = (float)raw.pl, S = (float)raw.ol;
  const float De = fmaf(S, cr.Db, cr.Dt);
  RequestSide q;
  q.u = make_float4(L, live ? cr.Dt : -1.0f, live ? cr.Db : -1.0f, S);
  q.w = make_float4(cr.iDt, cr.iDb, De, 1.0f / De);
  return q;
}

// One candidate's results: its admitted requests and, with kScore, the composite score - Phi = alpha * Phi_S^n +
// beta * min(Phi_T, gamma_T) / gamma_T + (1 - beta) * max(gamma_L - Phi_L, 0) / gamma_L (Sec. IV-D, Eq. 6-8).
template <bool kScore>
__device__ __forceinline__ void write_candidate(const SweepWindowArgs& a, const SweepWindowSet& rs, uint32_t c,
                                                uint32_t sat, unsigned long long wait_sum, float pt) {
  rs.sat_count[c] = sat;
  if (!kScore) return;
  const float ps = (rs.n_req == 0u) ? 0.0f : (float)sat / (float)rs.n_req;
  const float pl = (sat == 0u) ? 0.0f : ((float)wait_sum * 0x1p-20f) / (float)sat;
  const float ptn = fminf(pt, a.gamma_t) / a.gamma_t;
  const float pln = fmaxf(a.gamma_l - pl, 0.0f) / a.gamma_l;
  const float sc = fmaf(a.alpha, ps, fmaf(a.beta, ptn, (1.0f - a.beta) * pln));
  if (rs.phi_s) rs.phi_s[c] = ps;
  if (rs.phi_t) rs.phi_t[c] = pt;
  if (rs.phi_l) rs.phi_l[c] = pl;
  if (rs.score) rs.score[c] = sc;
}

// Scores V requests of a lane against M <= kFew instances held in registers and adds what is admitted
// to the caller's sums: cnt[i] (uniform) requests and acc[i] (per lane) prefill ticks on instance i, except
// that the entries of instance 0 take everything admitted (the caller subtracts the others).  Who is
// given what stays in lane masks on the scalar unit.  Needs AdmissionBounds::narrow.
constexpr int kFew = 4;
template <int M, int V, bool kSQ>
__device__ __forceinline__ void score_few(const SlotRecord (&r)[kFew], const float (&rank)[kFew],
                                          const RequestSide (&q)[V], uint32_t (&cnt)[kFew],
                                          unsigned long long (&acc)[kFew]) {
  static_assert(V <= 4, "V prefills of up to 2^29 ticks in 32 bits");
  uint32_t sum[M] = {};
#pragma unroll
  for (int v = 0; v < V; ++v) {
    float best, bpre;
    unsigned long long took[M];  // lanes whose best so far instance i is
    if (M == 1) {
      // one instance: only whether it is capable matters.  Its slack is >= 0 iff the first-token and
      // the between-token latency meet their deadlines (the end-to-end margin is implied by the two).
      bpre = fmaf(r[0].p, q[v].u.x, r[0].a);
      took[0] = lane_mask(r[0].wait + bpre <= q[v].u.y) & lane_mask(r[0].tbt <= q[v].u.z);
    } else {
      const Deadlines d{q[v].u.y, q[v].u.z, q[v].w.z, q[v].w.x, q[v].w.y, q[v].w.w};
#pragma unroll
      for (int i = 0; i < M; ++i) {
        const Margins m = score_triple(r[i].a, r[i].p, r[i].tbt, r[i].wait, q[v].u.x, q[v].u.w, d);
        const float val = (kSQ && m.slack >= 0.0f) ? rank[i] : m.slack;
        if (i == 0) {
          best = val;
          bpre = m.pre;
        } else {
          const bool better = val > best;
          took[i] = lane_mask(better);
          bpre = better ? m.pre : bpre;
          best = max_no_nan(best, val);
        }
      }
      // admitted requests load their instance; of two takers the later one holds the request
      unsigned long long left = lane_mask(best >= 0.0f);
      took[0] = left;
#pragma unroll
      for (int i = M - 1; i > 0; --i) {
        took[i] &= left;
        left &= ~took[i];
      }
    }
    const uint32_t ticks = (uint32_t)rintf(bpre * 1048576.0f);
#pragma unroll
    for (int i = 0; i < M; ++i) {
      cnt[i] += (uint32_t)__popcll(took[i]);
      sum[i] += in_mask(took[i]) ? ticks : 0u;
    }
  }
#pragma unroll
  for (int i = 0; i < M; ++i) acc[i] += sum[i];
}

// kScore: also observe what the composite serving score needs (Sec. IV-D, Eq. 6-8) - which instances
// served a request, and the exact integer sum of the admitted requests' queue waits - and finish the
// candidate's score: Phi = alpha * Phi_S^n + beta * min(Phi_T, gamma_T) / gamma_T +
// (1 - beta) * max(gamma_L - Phi_L, 0) / gamma_L with Phi_T = sum of 1 / tbt_j over the serving
// instances in index order (tbt_j of the first window) and Phi_L = mean wait of the admitted requests.
// S: instance slots per lane, instance j = s * 64 + lane.
// NW = 1: a wavefront owns a candidate.  The four of a block score the same requests, so a chunk of 256
// is fetched and prepared once per block (a request per thread) and read by all from LDS.
// NW = 4: the wavefronts of a block share a candidate.  Each keeps the whole state and advances it by
// itself; the requests of a window are dealt among them, V per lane at a time, and the admitted sums
// meet in LDS behind the window's only barrier.
// kSQ: the distributor's shortest-queue rule instead of the largest slack.
template <bool kScore, int S, int NW, int V, bool kSQ>
__global__ __launch_bounds__(kAssignThreads, S <= 2 ? 4 : 3) void sweep_window_kernel(const SweepWindowArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* tab = reinterpret_cast<float*>(smem);
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ float4 chunk_u[NW == 1 ? 2 : 1][NW == 1 ? kAssignThreads : 1];  // RequestSide in two arrays:
  __shared__ float4 chunk_w[NW == 1 ? 2 : 1][NW == 1 ? kAssignThreads : 1];  // no bank conflicts
  // admitted sums of a window.  NW > 1: three buffers in turn - one is added to, the one before is read, the
  // one after is cleared.  NW = 1: one per wavefront, for windows with more than a few instances.
  constexpr uint32_t kSums = NW > 1 ? kSumBuffers : kAssignThreads / 64;
  __shared__ uint32_t n_sum[kSums][64 * S];
  __shared__ unsigned long long t_sum[kSums][64 * S];

  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  if (tid < a.n_slo) cls[tid] = ClassRow{a.d_ttft[tid], a.d_tbt[tid], a.i_ttft[tid], a.i_tbt[tid]};
  for (uint32_t i = tid; i < 3u * a.cells; i += kAssignThreads) tab[i] = a.tab[i];
  for (uint32_t i = tid; i < kSums * 64u * S; i += kAssignThreads) { (&n_sum[0][0])[i] = 0u; (&t_sum[0][0])[i] = 0ull; }
  __syncthreads();

  // blocks of one request set first, then the next: a block never mixes sets
  constexpr uint32_t kPerBlock = (uint32_t)(kAssignThreads / 64) / (uint32_t)NW;  // candidates
  const uint32_t blocks_per_set = (a.n_cand + kPerBlock - 1u) / kPerBlock;
  const uint32_t set = blockIdx.x / blocks_per_set;
  const uint32_t c = (blockIdx.x - set * blocks_per_set) * kPerBlock + (NW == 1 ? wave : 0u);
  const bool mine_c = c < a.n_cand;  // a block's last wavefronts may have no candidate: they only fetch
  const SweepWindowSet rs = resolve_set(a.sets[set]);
  const size_t base = (size_t)c * a.i_pad;
  const uint32_t n = mine_c ? min(a.n_inst[c], a.i_pad) : 0u;

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
  // queue waits of the admitted requests, in ticks: of windows with few instances (uniform), of the others (of
  // the lane's instances)
  unsigned long long wait_sum = 0ull, wait_own = 0ull;

  const uint32_t R = rs.n_req;
  auto window_end = [&](uint32_t s0) __attribute__((always_inline)) { return R - s0 > rs.window ? s0 + rs.window : R; };
  // Requests are fetched one batch ahead, across window boundaries: no window starts with a trip to
  // memory (two batches ahead: no faster).  A batch is 256 requests with NW = 1, 256 * V with NW = 4;
  // (f0, f1) is the next one to fetch and the end of the window it belongs to.  The arrival time that
  // passes behind a window is fetched one window ahead.
  constexpr uint32_t kRaw = NW == 1 ? 1u : (uint32_t)V;
  constexpr uint32_t kBatch = kAssignThreads * kRaw;
  RequestRaw raw[kRaw];
#pragma unroll
  for (uint32_t v = 0; v < kRaw; ++v) raw[v] = RequestRaw{0u, 0u, kNoRequest};
  uint32_t f0 = 0, f1 = window_end(0u);
  auto fetch = [&]() __attribute__((always_inline)) {
    if (f0 >= R) return;
#pragma unroll
    for (uint32_t v = 0; v < kRaw; ++v) raw[v] = fetch_request(rs, f0, v * kAssignThreads + tid, f1);
    if (f1 - f0 > kBatch) { f0 += kBatch; return; }
    f0 = f1;
    if (f0 < R) f1 = window_end(f0);
  };
  RequestSide rq[V];
  uint32_t cbuf = 0, buf = NW == 1 ? wave : 0u;
  auto next_chunk = [&](uint32_t to) __attribute__((always_inline)) {
    const RequestSide q = request_side(raw[0], a.n_slo, cls, a.status);
    chunk_u[to][NW == 1 ? tid : 0u] = q.u;
    chunk_w[to][NW == 1 ? tid : 0u] = q.w;
    fetch();
  };
  fetch();
  if (NW == 1) {  // the first chunk; the next is on its way
    next_chunk(0u);
    __syncthreads();
  }
  uint32_t t_begin = 0, t_end = 0;
  if (R > rs.window) { t_begin = rs.arrival_ticks[0]; t_end = rs.arrival_ticks[rs.window]; }

  for (uint32_t s0 = 0, e0 = 0; s0 < R; s0 = e0) {
    e0 = window_end(s0);
    uint32_t t_next = 0;  // when the window after the next one opens
    if (e0 < R && window_end(e0) < R) t_next = rs.arrival_ticks[window_end(e0)];
    SlotRecord rec[S];
    float svc[S];
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if ((uint32_t)s * 64u >= n && s != 0) continue;  // uniform: no instance in this row of slots
      unsigned long long bad;
      slot[s].stage(tab, a.cells, a.mp, rec[s], svc[s], bad);
      bad_slot |= bad;  // (a lane without an instance is never bad)
      if (kScore && s0 == 0u) inv_tbt_first[s] = in_mask(bad) ? 0.0f : 1.0f / rec[s].tbt;
    }

    // which instances a request can be admitted to at all in this window, and the first few of them
    InstanceSet<S> und;
    SlotRecord fr[kFew];
    uint32_t fj[kFew];
    int32_t focc[kFew];
    int32_t occ[S];  // as the window opens
#pragma unroll
    for (int s = 0; s < S; ++s) occ[s] = slot[s].occ;
    find_admissible<S, kSQ>(rec, occ, n, lane, a.bounds, und);
    const uint32_t m = und.count();
    const bool few = m <= (uint32_t)kFew && a.bounds.narrow;
    if (few) first_of<S, kSQ, kFew>(und, rec, occ, fr, fj, focc);
    float frank[kFew];
    uint32_t cnt[kFew];
    unsigned long long acc[kFew];
#pragma unroll
    for (int i = 0; i < kFew; ++i) { cnt[i] = 0u; acc[i] = 0ull; }
    float rank[S];
    if (kSQ) {
      if (few) {
#pragma unroll
        for (int i = 0; i < kFew; ++i) {
          uint32_t ahead = 0;
#pragma unroll
          for (int k = 0; k < kFew; ++k)
            ahead += ((uint32_t)k < m && (focc[k] < focc[i] || (focc[k] == focc[i] && k < i))) ? 1u : 0u;
          frank[i] = (float)(512u - ahead);
        }
      } else {
        queue_ranks<S>(occ, und, lane, rank);
      }
    }
    // adds to the state: instance j (uniform) admitted `num` requests of `ticks` prefill in all
    auto admit = [&](uint32_t j, uint32_t num, unsigned long long ticks, float wait) __attribute__((always_inline)) {
      if (kScore) wait_sum += (unsigned long long)num * to_ticks(wait, a.bounds.narrow);
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (j >> 6 == (uint32_t)s && (j & 63u) == lane) {
          slot[s].occ += (int32_t)num;
          slot[s].q += ticks;
          served[s] += num;
        }
    };
    // V requests per lane against the window's few instances
    auto score = [&](const RequestSide (&q)[V]) __attribute__((always_inline)) {
      if (m == 1u) score_few<1, V, kSQ>(fr, frank, q, cnt, acc);
      else if (m == 2u) score_few<2, V, kSQ>(fr, frank, q, cnt, acc);
      else if (m == 3u) score_few<3, V, kSQ>(fr, frank, q, cnt, acc);
      else if (m == 4u) score_few<4, V, kSQ>(fr, frank, q, cnt, acc);
    };
    // ... or against any number of them
    auto score_any = [&](const RequestSide (&q)[V]) __attribute__((always_inline)) {
      float best[V], bpre[V];
      uint32_t idx[V];
#pragma unroll
      for (int v = 0; v < V; ++v) { best[v] = -INFINITY; bpre[v] = 0.0f; idx[v] = 0xffffffffu; }
#pragma unroll
      for (int s = 0; s < S; ++s) {
        for (unsigned long long todo = und.m[s]; todo != 0ull; todo &= todo - 1ull) {
          const int l = (int)__builtin_ctzll(todo);
          const SlotRecord r = rec[s].of_lane(l);
          const float rk = kSQ ? lane_value(rank[s], l) : 0.0f;
#pragma unroll
          for (int v = 0; v < V; ++v) {
            const Deadlines d{q[v].u.y, q[v].u.z, q[v].w.z, q[v].w.x, q[v].w.y, q[v].w.w};
            const Margins mg = score_triple(r.a, r.p, r.tbt, r.wait, q[v].u.x, q[v].u.w, d);
            const float val = (kSQ && mg.slack >= 0.0f) ? rk : mg.slack;
            const bool better = val > best[v];
            idx[v] = better ? (uint32_t)(s * 64 + l) : idx[v];
            bpre[v] = better ? mg.pre : bpre[v];
            best[v] = max_no_nan(best[v], val);
          }
        }
      }
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const bool adm = best[v] >= 0.0f;  // admitted requests load their instance
        const unsigned long long am = lane_mask(adm);
        if (am == 0ull) continue;
        const unsigned long long ticks = adm ? to_ticks(bpre[v], a.bounds.narrow) : 0ull;
        const uint32_t one = (uint32_t)__builtin_amdgcn_readlane((int)idx[v], (int)__builtin_ctzll(am));
        if (lane_mask(adm && idx[v] == one) == am) {  // all chose one instance
          const unsigned long long tsum = wave_sum_ticks(ticks);
          if (lane == 0u) {
            atomicAdd(&n_sum[buf][one], (uint32_t)__popcll(am));
            atomicAdd(&t_sum[buf][one], tsum);
          }
        } else if (adm) {
          atomicAdd(&n_sum[buf][idx[v]], 1u);
          atomicAdd(&t_sum[buf][idx[v]], ticks);
        }
      }
    };
    // ... and what they were given, every lane for its instances
    auto close_any = [&](uint32_t from) __attribute__((always_inline)) {
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const uint32_t num = n_sum[from][s * 64 + lane];
        slot[s].occ += (int32_t)num;
        slot[s].q += t_sum[from][s * 64 + lane];
        served[s] += num;
        if (kScore && num != 0u) wait_own += (unsigned long long)num * to_ticks(rec[s].wait, a.bounds.narrow);
      }
    };
    auto close_few = [&]() __attribute__((always_inline)) {
      if (!few) return;
#pragma unroll
      for (int i = 1; i < kFew; ++i) { cnt[0] -= cnt[i]; acc[0] -= acc[i]; }
#pragma unroll
      for (int i = 0; i < kFew; ++i)
        if (cnt[i] != 0u) {
          const unsigned long long tsum = wave_sum_ticks(acc[i]);
          if (NW > 1) {
            if (lane == 0u) { atomicAdd(&n_sum[buf][fj[i]], cnt[i]); atomicAdd(&t_sum[buf][fj[i]], tsum); }
          } else {
            admit(fj[i], cnt[i], tsum, fr[i].wait);
          }
        }
    };

    if (NW == 1) {
      for (uint32_t b0 = s0; b0 < e0; b0 = e0 - b0 > kBatch ? b0 + kBatch : e0) {
        next_chunk(cbuf ^ 1u);  // the chunk after this one (past the end: nothing that counts)
        const uint32_t len = min(e0 - b0, kBatch);
        if (m != 0u) {
          for (uint32_t i0 = 0; i0 < len; i0 += 64u * V) {
#pragma unroll
            for (int v = 0; v < V; ++v) {
              const uint32_t i = i0 + (uint32_t)v * 64u + lane;
              rq[v] = RequestSide{chunk_u[cbuf][i], chunk_w[cbuf][i]};
            }
            if (few) score(rq);
            else score_any(rq);
          }
        }
        cbuf ^= 1u;
        __syncthreads();
      }
      if (few) {
        close_few();
      } else if (m != 0u) {  // a wavefront's own LDS operations stay in order
        __builtin_amdgcn_wave_barrier();
        close_any(buf);
#pragma unroll
        for (int s = 0; s < S; ++s) { n_sum[buf][s * 64 + lane] = 0u; t_sum[buf][s * 64 + lane] = 0ull; }
      }
    } else {
      for (uint32_t b0 = s0; b0 < e0; b0 = e0 - b0 > kBatch ? b0 + kBatch : e0) {
#pragma unroll
        for (int v = 0; v < V; ++v) rq[v] = request_side(raw[NW == 1 ? 0 : v], a.n_slo, cls, a.status);
        fetch();
        if (few) score(rq);
        else score_any(rq);
      }
      close_few();
      const uint32_t free = cleared_sum_buffer(buf);  // clean before anyone passes this barrier
      if (tid < 64u * S) { n_sum[free][tid] = 0u; t_sum[free][tid] = 0ull; }
      lds_atomics_barrier();
      if (few) {
#pragma unroll
        for (int i = 0; i < kFew; ++i)
          if ((uint32_t)i < m) admit(fj[i], n_sum[buf][fj[i]], t_sum[buf][fj[i]], fr[i].wait);
      } else {
        close_any(buf);
      }
      buf = next_sum_buffer(buf);
    }
    if (e0 < R) {  // time passes until the next window opens
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (s == 0 || (uint32_t)s * 64u < n) slot[s].advance(t_end - t_begin, svc[s]);
    }
    t_begin = t_end;
    t_end = t_next;
  }

  if (bad_slot != 0ull) raise_status(a.status, 2u);
  uint32_t sat = 0;
#pragma unroll
  for (int s = 0; s < S; ++s) sat += served[s];
  sat = wave_sum_u32(sat);
  float pt = 0.0f;
  if (kScore) {
    for (int d = 32; d >= 1; d >>= 1) wait_own += __shfl_xor(wait_own, d);
    wait_sum += wait_own;
    // Phi_T: 1 / tbt of the serving instances, added in index order
#pragma unroll
    for (int s = 0; s < S; ++s)
      for (unsigned long long todo = lane_mask(served[s] != 0u); todo != 0ull; todo &= todo - 1ull)
        pt = pt + lane_value(inv_tbt_first[s], (int)__builtin_ctzll(todo));
  }
  if (lane == 0u && mine_c && (NW == 1 || wave == 0u)) write_candidate<kScore>(a, rs, c, sat, wait_sum, pt);
}

// Best candidate by score: largest score, lowest index on ties.  One block.
__global__ __launch_bounds__(1024) void score_argmax_kernel(const float* __restrict__ score,
                                                            uint32_t n_cand,
                                                            uint32_t* __restrict__ best_cand) {
  __shared__ unsigned long long best[16];
  unsigned long long key = 0ull;  // (order-preserving bits of the score << 32) | ~index
  for (uint32_t c = threadIdx.x; c < n_cand; c += blockDim.x) {
    const uint32_t b = __float_as_uint(score[c]);
    const uint32_t ord = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
    const unsigned long long kc = ((unsigned long long)ord << 32) | (unsigned long long)(~c);
    key = kc > key ? kc : key;
  }
  for (int d = 32; d >= 1; d >>= 1) {
    const unsigned long long o = __shfl_xor(key, d);
    key = o > key ? o : key;
  }
  if ((threadIdx.x & 63u) == 0u) best[threadIdx.x >> 6] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (uint32_t w = 1; w < (blockDim.x >> 6); ++w) key = best[w] > key ? best[w] : key;
    *best_cand = ~(uint32_t)(key & 0xffffffffull);
  }
}

}  // namespace maaso
