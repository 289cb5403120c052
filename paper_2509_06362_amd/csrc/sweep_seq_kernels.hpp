// Capacity-aware evaluation of candidate deployments with SHORT windows, down to one request per
// window - where every request meets the state left by all earlier ones, the paper's simulator taken
// literally (Sec. V-A: requests are mapped to slots one after the other and instance clocks advance
// in between).
//
// With a handful of requests per window the lanes of sweep_window_kernel (lanes = requests) are
// mostly idle.  Here a candidate belongs to ONE wavefront and the lanes are its INSTANCES (S slots per
// lane, instance j = s * 64 + lane): state, profile evaluation, triple, and the drain between two windows
// all stay in the lane's registers and the best instance of a request is a DPP arg-max over the
// wavefront.  Requests come prepared (deadlines, the reciprocal of the end-to-end one) through LDS.
//
// An instance's profile evaluation depends on the requests on it alone, so it is redone only where they
// changed: for the row of slots that admitted a request, or for all of them in the rare window at whose
// end a request completes.  What every window needs is the queued prefill (one conversion, one fma per
// slot) and the comparison that shows that nothing completes (no division).  8192 candidates of 128
// instances, 8192 requests one by one: 23.4 -> 9.6 ms, bound by issue (89 vector and 46 scalar instructions
// a request, all told); one placement of 64 instances: 0.56 -> 0.36 us per request, the chain of one request
// after the other in a single wavefront (49 vector and 31 scalar instructions, eleven cycles each on average).
//
// The arithmetic is the windowed kernel's, operation by operation, so the two agree bit for bit and
// with the oracle's windowed distributor.  The shortest-queue rule is not offered here (its ranks
// need every instance's queue length); the windowed kernel serves it.
#pragma once

#include "sweep_window_kernels.hpp"
#include "window_kernels.hpp"
#include "window_rules.hpp"

#pragma clang fp contract(off)

namespace maaso {

constexpr int kSeqThreads = 256;  // four wavefronts = four candidates of a request set per block
constexpr uint32_t kSeqChunk = 64;  // requests prepared at a time, by one of the block's wavefronts in turn

// The three profile tables in LDS with one entry more each: the row of a slot without an instance, whose
// prefill time is infinite.
__device__ __forceinline__ void load_seq_tables(float* tab, const float* src, uint32_t cells) {
  for (uint32_t i = threadIdx.x; i < 3u * (cells + 1u); i += blockDim.x) {
    const uint32_t t = i / (cells + 1u), k = i - t * (cells + 1u);
    tab[i] = k < cells ? src[t * cells + k] : (t == 0u ? INFINITY : 1.0f);
  }
}

// A placement in the lanes of one wavefront, taken through windows of requests.
template <int S>
struct Sequence {
  LiveSlot slot[S];
  SlotRecord rec[S];  // as evaluated when the window opened
  float svc[S], past[S];
  float pre[S], slack[S];  // of the request scored last
  float ttft[S], e2e[S];
  unsigned long long bad;  // lanes with a slot outside the tables, over the whole run
  uint32_t dirty;          // rows of slots whose occupancy changed in this window
  bool wide;               // some queue holds 2^32 ticks or more

  __device__ __forceinline__ void load(int s, bool present, const ModelParams& mp, uint32_t cells, uint32_t tp,
                                       uint32_t b, int32_t occ, uint64_t q) {
    if (present) {
      slot[s].load(mp, tp, b, occ, q);
    } else {  // empty for good, on the extra row of the tables
      slot[s].clear();
      slot[s].row0 = cells - 1u;
    }
  }
  __device__ __forceinline__ void evaluate(int s, const float* tab, uint32_t cells, const ModelParams& mp) {
    unsigned long long b;
    slot[s].evaluate(tab, cells + 1u, mp, rec[s], svc[s], past[s], b);
    if (b != 0ull) {  // (see close_window: a slot with a negative occupancy compares with no number)
      rare_path();
      if (slot[s].occ < 0) svc[s] = __builtin_nanf("");
      bad |= b;
    }
  }
  __device__ __forceinline__ void begin(const float* tab, uint32_t cells, const ModelParams& mp) {
    bad = 0ull;
    dirty = 0u;
    wide = false;  // (an admission cannot make it true where narrow_queue holds)
#pragma unroll
    for (int s = 0; s < S; ++s) {
      evaluate(s, tab, cells, mp);
      wide |= slot[s].any_wide();
    }
  }
  __device__ __forceinline__ void open_window() {
#pragma unroll
    for (int s = 0; s < S; ++s) rec[s].wait = slot[s].wait_with(past[s], wide);
  }
  // Largest slack of the request over all instances, uniform: four DPP steps settle each row of 16 lanes,
  // two row broadcasts carry the rows' maxima into lane 63, one v_readlane fetches it.
  __device__ __forceinline__ float score(const RequestSide& q) {
    const Deadlines d{q.u.y, q.u.z, q.w.z, q.w.x, q.w.y, q.w.w};
    float m = -INFINITY;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const Margins g = score_triple(rec[s].a, rec[s].p, rec[s].tbt, rec[s].wait, q.u.x, q.u.w, d);
      pre[s] = g.pre;
      slack[s] = g.slack;
      ttft[s] = g.ttft;
      e2e[s] = g.e2e;
      m = s == 0 ? g.slack : max_no_nan(m, g.slack);
    }
    m = max_lanes<16>(m);
    MAASO_DPP_FOLD_ROWS("v_max_f32_dpp", m, "row_bcast:15", "0xa");
    MAASO_DPP_FOLD_ROWS("v_max_f32_dpp", m, "row_bcast:31", "0xc");
    return lane_value(m, 63);
  }
  // The lowest index among the instances whose slack is `best` (above -inf): the first row of slots with a
  // holder, its first lane, from one lane mask per row on the scalar unit.
  __device__ __forceinline__ uint32_t holder(float best) const {
    uint32_t j = 0;
#pragma unroll
    for (int s = S - 1; s >= 0; --s) {
      const unsigned long long held = lane_mask(slack[s] == best);
      if (held != 0ull) j = (uint32_t)s * 64u + (uint32_t)__builtin_ctzll(held);
    }
    return j;
  }
  // The request scored last is admitted to instance j = (s, l): it loads it at the window's end.
  __device__ __forceinline__ void admit(int s, uint32_t l, uint32_t lane, const bool narrow) {
    const bool me = l == lane;
    const unsigned long long t = to_ticks(pre[s], narrow);
    slot[s].occ += me ? 1 : 0;
    slot[s].q += me ? t : 0ull;
    if (!narrow) {
      rare_path();
      wide |= slot[s].any_wide();
    }
    dirty |= 1u << s;
  }
  // `delta` ticks pass (`last`: nothing follows, no time passes).
  __device__ __forceinline__ void close_window(uint32_t delta, bool last, const float* tab, uint32_t cells,
                                               const ModelParams& mp) {
    if (!last) {
      const float dt = (float)delta * 0x1p-20f;
      float served[S];
      unsigned long long some = 0ull;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const uint64_t before = slot[s].q;
        slot[s].q = (uint64_t)__builtin_elementwise_sub_sat((uint32_t)before, delta);
        if (wide) {
          rare_path();
          slot[s].q = before - (before < (uint64_t)delta ? before : (uint64_t)delta);
        }
        served[s] = (float)min(slot[s].occ, (int32_t)slot[s].B) * dt;
        some |= lane_mask(!(served[s] < svc[s]));
      }
      // 0 <= served < svc everywhere: the correctly rounded quotients are below one and nothing completes
      if (some != 0ull) {
        rare_path();
#pragma unroll
        for (int s = 0; s < S; ++s) {
          const float x = served[s] / (slot[s].occ < 0 ? 1.0f : svc[s]);
          slot[s].occ -= min(slot[s].occ, (int32_t)floorf(fminf(x, 2147483520.0f)));
        }
        dirty = (1u << S) - 1u;
      }
    }
    if (dirty != 0u) {
#pragma unroll
      for (int s = 0; s < S; ++s)
        if (dirty & (1u << s)) evaluate(s, tab, cells, mp);
      dirty = 0u;
    }
  }
};

// kOne: every set's window is one request (the window length is then a constant).
template <bool kScore, int S, bool kOne = false>
__global__ __launch_bounds__(kSeqThreads, S <= 2 ? 8 : 4) void sweep_seq_kernel(const SweepWindowArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* tab = reinterpret_cast<float*>(smem);
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ float4 chunk_u[2][kSeqChunk], chunk_w[2][kSeqChunk];  // RequestSide
  __shared__ uint32_t chunk_t[2][kSeqChunk];                       // arrival of the request behind it

  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  if (tid < a.n_slo) cls[tid] = ClassRow{a.d_ttft[tid], a.d_tbt[tid], a.i_ttft[tid], a.i_tbt[tid]};
  load_seq_tables(tab, a.tab, a.cells);
  __syncthreads();

  constexpr uint32_t kPerBlock = kSeqThreads / 64;
  const uint32_t blocks_per_set = (a.n_cand + kPerBlock - 1u) / kPerBlock;
  const uint32_t set = blockIdx.x / blocks_per_set;
  const uint32_t c = (blockIdx.x - set * blocks_per_set) * kPerBlock + wave;
  const bool mine_c = c < a.n_cand;  // a block's last wavefronts may have no candidate: they only prepare
  const SweepWindowSet rs = resolve_set(a.sets[set]);
  const size_t base = (size_t)c * a.i_pad;
  const uint32_t n = mine_c ? min(a.n_inst[c], a.i_pad) : 0u;

  Sequence<S> sq;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    uint32_t tp = 0, B = 1;
    int32_t occ = 0;
    uint64_t q = 0;
    if (j < n) { tp = a.tp_idx[base + j]; B = a.max_batch[base + j]; occ = a.occ[base + j]; q = a.q_ticks[base + j]; }
    sq.load(s, j < n, a.mp, a.cells, tp, B, occ, q);
  }
  sq.begin(tab, a.cells, a.mp);
  unsigned long long served[S];
  float inv_tbt_first[S];
#pragma unroll
  for (int s = 0; s < S; ++s) {
    served[s] = 0ull;
    inv_tbt_first[s] = kScore ? (in_mask(sq.bad) && sq.past[s] == INFINITY ? 0.0f : 1.0f / sq.rec[s].tbt) : 0.0f;
  }
  uint32_t sat = 0;                    // uniform
  unsigned long long wait_sum = 0ull;  // queue waits of the admitted requests, in ticks; uniform

  const uint32_t R = rs.n_req;
  const uint32_t W = kOne ? 1u : rs.window;
  // Chunk k is prepared by wavefront k mod 4 from what it asked for four chunks earlier.
  uint32_t f0 = wave * kSeqChunk;
  RequestRaw raw{0u, 0u, kNoRequest};
  uint32_t behind = 0;
  auto fetch = [&]() __attribute__((always_inline)) {
    if (f0 >= R) return;
    raw = fetch_request(rs, f0, lane, R);
    if (reads_arrival_behind(f0 + lane, R, W)) behind = rs.arrival_ticks[f0 + lane + 1u];
    f0 = R - f0 > 4u * kSeqChunk ? f0 + 4u * kSeqChunk : R;
  };
  auto prepare = [&](uint32_t to) __attribute__((always_inline)) {
    const RequestSide q = request_side(raw, a.n_slo, cls, a.status);
    chunk_u[to][lane] = q.u;
    chunk_w[to][lane] = q.w;
    chunk_t[to][lane] = behind;
    fetch();
  };
  fetch();
  if (wave == 0u) prepare(0u);
  __syncthreads();

  uint32_t t_open = R > W ? rs.arrival_ticks[0] : 0u;
  uint32_t in_window = 0;
  for (uint32_t c0 = 0, k = 0; c0 < R; ++k) {
    const uint32_t len = min(R - c0, kSeqChunk);
    const uint32_t buf = k & 1u;
    if (((k + 1u) & 3u) == wave && R - c0 > kSeqChunk) prepare(buf ^ 1u);
    for (uint32_t i = 0; i < len; ++i) {
      if (kOne || in_window == 0u) sq.open_window();
      const RequestSide q{chunk_u[buf][i], chunk_w[buf][i]};
      const float best = sq.score(q);
      if (best >= 0.0f) {  // admitted
        const uint32_t j = sq.holder(best), l = j & 63u;
        sat += 1u;
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (j >> 6 == (uint32_t)s) {
            rare_path();  // (a branch per row of slots, not selects over all of them)
            if (kScore) {
              served[s] |= 1ull << l;
              wait_sum += to_ticks(lane_value(sq.rec[s].wait, (int)l), a.bounds.narrow);
            }
            sq.admit(s, l, lane, a.bounds.narrow_queue);
          }
      }
      const bool last = c0 + i + 1u == R;
      if (kOne || ++in_window == W || last) {
        const uint32_t t_end = chunk_t[buf][i];
        sq.close_window(t_end - t_open, last, tab, a.cells, a.mp);
        t_open = t_end;
        in_window = 0u;
      }
    }
    c0 = R - c0 > kSeqChunk ? c0 + kSeqChunk : R;
    __syncthreads();
  }

  // results of this (set, candidate): lane 0 writes them
  if (sq.bad != 0ull && R != 0u) raise_status(a.status, 2u);  // (a lane without an instance is never bad)
  float pt = 0.0f;
  if (kScore) {
    // Phi_T: 1 / tbt of the serving instances, added in index order
#pragma unroll
    for (int s = 0; s < S; ++s)
      for (unsigned long long todo = served[s]; todo != 0ull; todo &= todo - 1ull)
        pt = pt + lane_value(inv_tbt_first[s], (int)__builtin_ctzll(todo));
  }
  if (lane == 0u && mine_c) write_candidate<kScore>(a, rs, c, sat, wait_sum, pt);
}

// The distributor itself on short windows (one placement, requests in arrival order, down to one
// request per window - the online distributor of Sec. IV-F taken literally): the same wavefront
// scheme, plus the per-request outputs.  One wavefront does all the work - the method is sequential
// here - so this is about latency: no device-wide barrier per window.  The outputs of 64 requests are
// collected one lane each and stored together.
template <bool kLat, int S>
__global__ __launch_bounds__(64) void assign_seq_kernel(const AssignArgs a, uint32_t window) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* tab = reinterpret_cast<float*>(smem);
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ float4 chunk_u[kSeqChunk], chunk_w[kSeqChunk];  // RequestSide
  __shared__ uint32_t chunk_t[kSeqChunk];                    // arrival of the request behind it
  const uint32_t lane = threadIdx.x;
  if (lane < a.n_slo) cls[lane] = ClassRow{a.d_ttft[lane], a.d_tbt[lane], a.i_ttft[lane], a.i_tbt[lane]};
  load_seq_tables(tab, a.tab, a.cells);
  __syncthreads();

  const PlacementRow row = select_row(a);
  const uint32_t n = row.n;
  Sequence<S> sq;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    uint32_t tp = 0, B = 1;
    int32_t occ = 0;
    uint64_t q = 0;
    if (j < n) { tp = row.tp_idx[j]; B = row.max_batch[j]; occ = row.occ[j]; q = row.q_ticks[j]; }
    sq.load(s, j < n, a.mp, a.cells, tp, B, occ, q);
  }
  sq.begin(tab, a.cells, a.mp);
  unsigned long long sat = 0ull;  // uniform

  const uint32_t R = a.n_req;
  const uint32_t W = window;
  auto fetch = [&](uint32_t c0, RequestRaw& raw, uint32_t& behind) __attribute__((always_inline)) {
    const uint32_t r = c0 + lane;
    raw = RequestRaw{0u, 0u, kNoRequest};
    if (r < R) { raw.pl = a.prompt_len[r]; raw.ol = a.out_len[r]; raw.k = a.slo_class[r]; }
    if (r + 1u < R) behind = a.arrival_ticks[r + 1u];
  };
  RequestRaw raw;
  uint32_t behind = 0;
  fetch(0u, raw, behind);
  uint32_t t_open = R > W ? a.arrival_ticks[0] : 0u;
  uint32_t in_window = 0;
  const float nanv = __builtin_nanf("");
  for (uint32_t c0 = 0; c0 < R; c0 = R - c0 > kSeqChunk ? c0 + kSeqChunk : R) {
    const uint32_t len = min(R - c0, kSeqChunk);
    // one wavefront: its LDS operations stay in order, no barrier between the writes and the reads
    const unsigned long long live = lane_mask(raw.k < a.n_slo);
    const RequestSide mine = request_side(raw, a.n_slo, cls, a.status);
    chunk_u[lane] = mine.u;
    chunk_w[lane] = mine.w;
    chunk_t[lane] = behind;
    if (R - c0 > kSeqChunk) fetch(c0 + kSeqChunk, raw, behind);
    // outputs of the chunk, request c0 + lane in this lane
    int32_t o_idx = -1;
    float o_slack = -INFINITY, o_ttft = nanv, o_tbt = nanv, o_e2e = nanv;
    for (uint32_t i = 0; i < len; ++i) {
      if (in_window == 0u) sq.open_window();
      const RequestSide q{chunk_u[i], chunk_w[i]};
      if ((live >> i) & 1ull) {
        const float best = sq.score(q);
        if (best > -INFINITY) {
          const uint32_t j = sq.holder(best);
          const bool me = lane == i;
          o_idx = me ? (int32_t)j : o_idx;
          o_slack = me ? best : o_slack;
          if (kLat) {  // what is reported about the chosen instance comes from the lane that holds it
#pragma unroll
            for (int s = 0; s < S; ++s)
              if (j >> 6 == (uint32_t)s) {
                const int l = (int)(j & 63u);
                const float w_ttft = lane_value(sq.ttft[s], l), w_tbt = lane_value(sq.rec[s].tbt, l),
                            w_e2e = lane_value(sq.e2e[s], l);
                o_ttft = me ? w_ttft : o_ttft;
                o_tbt = me ? w_tbt : o_tbt;
                o_e2e = me ? w_e2e : o_e2e;
              }
          }
          if (best >= 0.0f) {  // admitted: it loads the instance; a blocked request does not
            sat += 1ull;
#pragma unroll
            for (int s = 0; s < S; ++s)
              if (j >> 6 == (uint32_t)s) {
                rare_path();
                sq.admit(s, j & 63u, lane, a.bounds.narrow_queue);
              }
          }
        }
      }
      const bool last = c0 + i + 1u == R;
      if (++in_window == W || last) {
        const uint32_t t_end = chunk_t[i];
        sq.close_window(t_end - t_open, last, tab, a.cells, a.mp);
        t_open = t_end;
        in_window = 0u;
      }
    }
    const uint32_t mine_r = c0 + lane;
    if (mine_r < R) {
      if (a.chosen) a.chosen[mine_r] = o_idx;
      if (a.slack) a.slack[mine_r] = o_slack;
      if (kLat) {
        if (a.ttft) a.ttft[mine_r] = o_ttft;
        if (a.tbt) a.tbt[mine_r] = o_tbt;
        if (a.e2e) a.e2e[mine_r] = o_e2e;
      }
    }
  }
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    if (j < n) { row.occ[j] = sq.slot[s].occ; row.q_ticks[j] = sq.slot[s].q; }
  }
  if (sq.bad != 0ull) raise_status(a.status, 2u);
  if (lane == 0u && a.n_satisfied) *a.n_satisfied = sat;
}

}  // namespace maaso
