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
// changed.  What every window needs is the queued prefill (one conversion, one fma per slot) and one
// comparison that shows that nothing completes (no division).
//
// What bounds it: vector issue, with eight wavefronts per SIMD.  Measured there, cycles per wavefront
// instruction: fma, add, sub, mul, mov, 32-bit add and saturating sub 2.3; all others - compare, convert,
// min, DPP, lane reads and writes, anything with a scalar operand - 4.2, scalar instructions about 2 beside them.  So the
// rules of NarrowSequence leave out conversions and compares first.  8192 candidates of 128 instances, 8192
// requests one by one: 23.4 -> 9.5 ms with the profile evaluated where occupancy changed -> 6.1 ms with 32-bit queues
// throughout, one lane evaluated per admission and the completion check on the scalar unit (93 -> 62 vector and 49 -> 29
// scalar instructions a request); 1000 requests, 6000 x 60 slots, windows of 3: 453 -> 385 us; 9000 x 128, of 16: 798 -> 593 us.
// Reading the next request ahead of its turn
// costs its registers' moves: 8 candidates 446 -> 429 us, 16,384 902 -> 1013 us; not taken.
//
// A block has one form for all of its candidates (they meet at barriers while they prepare requests): one slot that does not
// fit - 2^32 ticks queued, a negative occupancy, outside the tables - puts all four or eight on the general one.  With one
// such slot in every eighth candidate and in each, 3000 candidates, windows of 3, us: 16 slots 63 -> 68 -> 69, 128: 87 -> 96 -> 99.
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

constexpr int kSeqThreads = 512;    // up to eight wavefronts = candidates of a request set per block
constexpr uint32_t kSeqLds = 160u << 10;  // LDS of a compute unit
constexpr uint32_t kSeqChunk = 64;  // requests prepared at a time, by one of the block's wavefronts in turn

// The three profile tables in LDS, a row {a, p, tbt, row_safe_ticks} per entry, and one row more: that of a
// slot without an instance, whose prefill time is infinite and where nothing ever completes.
__device__ __forceinline__ void load_seq_rows(float4* rows, const float* src, uint32_t cells, const ModelParams& mp,
                                              uint32_t window) {
  for (uint32_t i = threadIdx.x; i <= cells; i += blockDim.x) {
    float4 r = make_float4(INFINITY, 1.0f, 1.0f, __uint_as_float(0xffffffffu));
    if (i < cells) {
      const float tbt = src[2u * cells + i];
      r = make_float4(src[i], src[cells + i], tbt,
                      __uint_as_float(row_safe_ticks(mp.s_bar, tbt, i % (mp.b_cap + 1u), window)));
    }
    rows[i] = r;
  }
}

// The request scored against every slot of the lane, and the largest slack over all instances, uniform: four DPP
// steps settle each row of 16 lanes, two row broadcasts carry the rows' maxima into lane 63, one v_readlane
// fetches it.
template <int S>
__device__ __forceinline__ float score_slots(const RequestSide& q, const SlotRecord (&rec)[S], float (&pre)[S],
                                             float (&slack)[S], float (&ttft)[S], float (&e2e)[S]) {
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
template <int S>
__device__ __forceinline__ uint32_t holder_of(const float (&slack)[S], float best) {
  uint32_t j = 0;
#pragma unroll
  for (int s = S - 1; s >= 0; --s) {
    const unsigned long long held = lane_mask(slack[s] == best);
    if (held != 0ull) j = (uint32_t)s * 64u + (uint32_t)__builtin_ctzll(held);
  }
  return j;
}

// A placement in the lanes of one wavefront, taken through windows of requests.
// kFits: narrow_queue holds, so that no admission makes `wide` true and a prefill's ticks fit 32 bits (false is always
// right).
template <int S, bool kFits>
struct Sequence {
  static constexpr bool kNarrow = false;
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
  __device__ __forceinline__ void evaluate(int s, const float4* rows, const ModelParams& mp) {
    unsigned long long b;
    slot[s].template evaluate<4u>(reinterpret_cast<const float*>(rows), 1u, mp, rec[s], svc[s], past[s], b);
    if (b != 0ull) {  // (see close_window: a slot with a negative occupancy compares with no number)
      rare_path();
      if (slot[s].occ < 0) svc[s] = __builtin_nanf("");
      bad |= b;
    }
  }
  __device__ __forceinline__ void begin(const float4* rows, const ModelParams& mp) {
    bad = 0ull;
    dirty = 0u;
    wide = false;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      evaluate(s, rows, mp);
      wide |= slot[s].any_wide();
    }
  }
  __device__ __forceinline__ void open_window() {
#pragma unroll
    for (int s = 0; s < S; ++s) rec[s].wait = slot[s].wait_with(past[s], wide);
  }
  __device__ __forceinline__ int32_t occupancy(int s) const { return slot[s].occ; }
  __device__ __forceinline__ uint64_t queue(int s) const { return slot[s].q; }
  // The request scored last is admitted to instance j = (s, l): it loads it at the window's end.
  template <bool kOne>
  __device__ __forceinline__ void admit(int s, uint32_t l, const float4*, const ModelParams&) {
    const bool me = in_mask(1ull << l);
    const unsigned long long t = to_ticks(pre[s], kFits);
    slot[s].occ += me ? 1 : 0;
    slot[s].q += me ? t : 0ull;
    if (!kFits) wide |= slot[s].any_wide();
    dirty |= 1u << s;
  }
  // `delta` ticks pass (`last`: nothing follows, no time passes).
  template <bool kOne>
  __device__ __forceinline__ void close_window(uint32_t delta, uint32_t, bool last, const float4* rows, const ModelParams& mp) {
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
        if (dirty & (1u << s)) evaluate(s, rows, mp);
      dirty = 0u;
    }
  }
};

// The same placement where nothing needs 64 bits and every slot is inside the tables: the usual case, for which a
// request costs some three fifths of what it costs above.  Queues are 32 bits.  What follows from an
// instance's occupancy is evaluated for the one lane that admitted a request.  Whether a request completes
// at a window's end is one comparison per row of slots with a number of ticks in which none can
// (row_safe_ticks), with windows of one request a single scalar one with the least of them, kept as instances
// fill up.
template <int S>
struct NarrowSequence {
  static constexpr bool kNarrow = true;
  uint32_t row0[S];        // byte offset of its strategy's first row
  uint32_t B[S];           // batch cap
  float invB[S];
  uint32_t arr[S];         // requests on it, an arriving one included
  uint32_t q[S];
  SlotRecord rec[S];       // as evaluated when the window opened
  float past[S];
  uint32_t safe[S];
  float pre[S], slack[S];  // of the request scored last
  float ttft[S], e2e[S];
  unsigned long long changed[S];  // lanes that admitted a request in this window
  uint32_t safe_all, safe_next;   // windows of one request: the least of all, now and once the window has closed

  // Whether a slot may be kept this way (`extra`: requests of the run).
  __device__ __forceinline__ static bool fits(const ModelParams& mp, uint32_t tp, uint32_t b, int32_t occ, uint64_t q,
                                              uint32_t extra) {
    return tp < mp.n_tp && b != 0u && b <= mp.b_cap && occ >= 0 && occ < (1 << 30) && extra < (1u << 30) && (q >> 32) == 0ull;
  }
  __device__ __forceinline__ void load(int s, bool present, const ModelParams& mp, uint32_t cells, uint32_t tp,
                                       uint32_t b, int32_t o, uint64_t ticks) {
    row0[s] = 16u * (present ? tp * (mp.b_cap + 1u) : cells - 1u);  // (an empty slot: on the extra row for good)
    B[s] = present ? b : 1u;
    invB[s] = 1.0f / (float)B[s];
    arr[s] = present ? (uint32_t)o + 1u : 1u;
    q[s] = present ? (uint32_t)ticks : 0u;
    changed[s] = 0ull;
  }
  // The table row, and with the occupancy penalty the latency per token, of slot s with `load` requests on it.
  __device__ __forceinline__ uint32_t batch(int s, uint32_t load, const ModelParams& mp) const {
    return min(load | (0u - mp.tbt_mode), B[s]);  // (worst-case latencies: any number, so the cap)
  }
  __device__ __forceinline__ float4 row(int s, uint32_t w, const float4* rows) const {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const unsigned char*>(rows) + (row0[s] + (w << 4)));
  }
  __device__ __forceinline__ float penalised(int s, float tbt, uint32_t w, const ModelParams& mp) const {
    const float over = (float)__builtin_elementwise_sub_sat(4u * w, 3u * B[s]);  // > 0 iff the batch is > 75 % full
    return tbt * fmaf(mp.pen_kappa, over * invB[s], 1.0f);
  }
  __device__ __forceinline__ void evaluate(int s, const float4* rows, const ModelParams& mp) {
    const uint32_t w = batch(s, arr[s], mp);
    const float4 r = row(s, w, rows);
    rec[s].a = r.x;
    rec[s].p = r.y;
    rec[s].tbt = r.z;
    if (mp.pen_kappa != 0.0f) {  // a factor of exactly one without a penalty
      rare_path();
      rec[s].tbt = penalised(s, r.z, w, mp);
    }
    safe[s] = __float_as_uint(r.w);
    const float ov = (float)__builtin_elementwise_sub_sat(arr[s], B[s]);  // requests beyond the batch cap
    past[s] = (ov * invB[s]) * (mp.s_bar * rec[s].tbt);
  }
  // All rows, and the least of the ticks in which nothing completes.
  __device__ __forceinline__ void begin(const float4* rows, const ModelParams& mp) {
    uint32_t least = 0xffffffffu;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      evaluate(s, rows, mp);
      least = min(least, safe[s]);
    }
    safe_all = safe_next = (uint32_t)__builtin_amdgcn_readfirstlane((int)min_lanes<64>(least));
  }
  __device__ __forceinline__ void open_window() {
#pragma unroll
    for (int s = 0; s < S; ++s) rec[s].wait = fmaf((float)q[s], 0x1p-20f, past[s]);
  }
  __device__ __forceinline__ int32_t occupancy(int s) const { return (int32_t)(arr[s] - 1u); }
  __device__ __forceinline__ uint64_t queue(int s) const { return q[s]; }
  // The request scored last is admitted to instance (s, l).  With windows of one request the instance is
  // evaluated for the next one right away.
  template <bool kOne>
  __device__ __forceinline__ void admit(int s, uint32_t l, const float4* rows, const ModelParams& mp) {
    changed[s] |= 1ull << l;
    if (in_mask(1ull << l)) {
      q[s] += (uint32_t)rintf(pre[s] * 1048576.0f);
      arr[s] += 1u;
      if (kOne) evaluate(s, rows, mp);
    }
    if (kOne) safe_next = min(safe_next, (uint32_t)__builtin_amdgcn_readlane((int)safe[s], (int)l));
  }
  // Requests complete, or may: the whole rule, against the service times that the window opened with.
  template <bool kOne>
  __device__ __forceinline__ void complete(uint32_t delta, const float4* rows, const ModelParams& mp) {
    const float dt = (float)delta * 0x1p-20f;
#pragma unroll
    for (int s = 0; s < S; ++s) {
      if (kOne) {  // the admitting lane is a request ahead
        const uint32_t one = in_mask(changed[s]) ? 1u : 0u;
        arr[s] -= one;
        evaluate(s, rows, mp);
        arr[s] += one;
      }
      const int32_t occ = (int32_t)(arr[s] - 1u);
      const float x = ((float)min(occ, (int32_t)B[s]) * dt) / (mp.s_bar * rec[s].tbt);
      arr[s] -= (uint32_t)min(occ, (int32_t)floorf(fminf(x, 2147483520.0f)));
      changed[s] = 0ull;
    }
    begin(rows, mp);
  }
  // `delta` ticks pass, none behind the last window, where nothing completes (narrow_queue: no service time is zero);
  // `at_most`: uniform, no fewer than those.
  template <bool kOne>
  __device__ __forceinline__ void close_window(uint32_t delta, uint32_t at_most, bool, const float4* rows, const ModelParams& mp) {
    if (kOne) {
#pragma unroll
      for (int s = 0; s < S; ++s) q[s] = __builtin_elementwise_sub_sat(q[s], delta);
      if (at_most >= safe_all && (uint32_t)__builtin_amdgcn_readfirstlane((int)delta) >= safe_all) {
        rare_path();
        complete<kOne>(delta, rows, mp);
      } else {
#pragma unroll
        for (int s = 0; s < S; ++s) changed[s] = 0ull;
        safe_all = safe_next;
      }
    } else {
      unsigned long long some = 0ull;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        some |= lane_mask(delta >= safe[s]);
        q[s] = __builtin_elementwise_sub_sat(q[s], delta);
      }
      if (some != 0ull) {
        rare_path();
        complete<kOne>(delta, rows, mp);
      } else {
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (changed[s] != 0ull) {
            rare_path();
            if (in_mask(changed[s])) evaluate(s, rows, mp);
            changed[s] = 0ull;
          }
      }
    }
  }
};

// What a block's wavefronts share while they walk through a request set: two chunks of requests, and with windows
// of one request the time behind each, else its arrival.
struct SeqChunks {
  float4 u[2][kSeqChunk], w[2][kSeqChunk];  // RequestSide
  uint32_t t[2][kSeqChunk];
  uint32_t t_max[2];  // kOne: the longest of a chunk's times
};
constexpr uint32_t kSeqShared = sizeof(SeqChunks) + kMaxSlo * sizeof(ClassRow);  // of a block beside the tables

// One candidate through the windows of a request set.  served: per row of slots, the lanes that admitted a
// request.  Every wavefront of the block calls it for the same set: they prepare the chunks in turn.
// kOne: the window is one request (a constant).
template <bool kScore, int S, bool kOne, class Seq>
__device__ __forceinline__ void walk_windows(const SweepWindowArgs& a, const SweepWindowSet& rs, Seq& sq,
                                             const float4* rows, const ClassRow* cls, SeqChunks& chunks, uint32_t lane,
                                             uint32_t wave, uint32_t n_waves, unsigned long long (&served)[S],
                                             uint32_t& sat, unsigned long long& wait_sum) {
  const uint32_t R = rs.n_req;
  const uint32_t W = kOne ? 1u : rs.window;
  // Chunk k is prepared by wavefront k mod n_waves from what it asked for n_waves chunks earlier.
  uint32_t f0 = wave * kSeqChunk, turn = wave;
  RequestRaw raw{0u, 0u, kNoRequest};
  uint32_t own = 0, behind = 0;
  auto fetch = [&]() __attribute__((always_inline)) {
    if (f0 >= R) return;
    raw = fetch_request(rs, f0, lane, R);
    own = behind = 0u;
    if (reads_arrival_behind(f0 + lane, R, W)) {
      behind = rs.arrival_ticks[f0 + lane + 1u];
      if (kOne) own = rs.arrival_ticks[f0 + lane];
    }
    f0 = R - f0 > n_waves * kSeqChunk ? f0 + n_waves * kSeqChunk : R;
  };
  auto prepare = [&](uint32_t to) __attribute__((always_inline)) {
    const RequestSide q = request_side(raw, a.n_slo, cls, a.status);
    chunks.u[to][lane] = q.u;
    chunks.w[to][lane] = q.w;
    chunks.t[to][lane] = kOne ? behind - own : behind;
    if (kOne) {
      const uint32_t top = ~min_lanes<64>(~(behind - own));
      if (lane == 0u) chunks.t_max[to] = top;
    }
    fetch();
  };
  fetch();
  if (wave == 0u) prepare(0u);
  __syncthreads();

  uint32_t t_open = !kOne && R > W ? rs.arrival_ticks[0] : 0u;
  uint32_t in_window = 0;
  for (uint32_t c0 = 0, buf = 0; c0 < R; buf ^= 1u) {
    const uint32_t len = min(R - c0, kSeqChunk);
    turn = turn == 0u ? n_waves - 1u : turn - 1u;  // how many chunks until this wavefront's turn
    if (turn == 0u && R - c0 > kSeqChunk) prepare(buf ^ 1u);
    const uint32_t at_most = kOne ? (uint32_t)__builtin_amdgcn_readfirstlane((int)chunks.t_max[buf]) : 0xffffffffu;
    unsigned long long admitted = 0ull;  // requests of the chunk, and (lane i) the wait of request i
    int waits = 0;
    unsigned long long bit = 1ull;
    auto one_request = [&](const RequestSide& q, uint32_t i) __attribute__((always_inline)) {
      const float best = score_slots<S>(q, sq.rec, sq.pre, sq.slack, sq.ttft, sq.e2e);
      // (a slack is no number or minus zero under no input: its between-token margin is a number, and a
      // difference from a deadline is +0 or far above the underflow)
      if (__builtin_bit_cast(int, best) >= 0) {
        const uint32_t j = holder_of<S>(sq.slack, best), l = j & 63u;
        admitted |= bit;
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (j >> 6 == (uint32_t)s) {
            rare_path();  // (a branch per row of slots, not selects over all of them)
            if (kScore) {
              served[s] |= 1ull << l;
              waits = with_lane(waits, (int)i, lane_value(sq.rec[s].wait, (int)l));
            }
            sq.template admit<kOne>(s, l, rows, a.mp);
          }
      }
      bit <<= 1;
    };
    if (kOne) {
      for (uint32_t i = 0; i < len; ++i) {
        const uint32_t passed = chunks.t[buf][i];
        sq.open_window();
        one_request(RequestSide{chunks.u[buf][i], chunks.w[buf][i]}, i);
        sq.template close_window<true>(passed, at_most, c0 + i + 1u == R, rows, a.mp);
      }
    } else {
      for (uint32_t i = 0; i < len;) {
        if (in_window == 0u) sq.open_window();
        const uint32_t stop = min(len, i + (W - in_window));  // of the window's requests in this chunk
        in_window += stop - i;
        do one_request(RequestSide{chunks.u[buf][i], chunks.w[buf][i]}, i);
        while (++i < stop);
        const bool last = c0 + stop == R;
        if (in_window == W || last) {
          const uint32_t t_end = chunks.t[buf][stop - 1u];
          sq.template close_window<false>(last ? 0u : t_end - t_open, at_most, last, rows, a.mp);
          t_open = t_end;
          in_window = 0u;
        }
      }
    }
    sat += (uint32_t)__popcll(admitted);
    if (kScore)
      wait_sum += wave_sum_ticks(in_mask(admitted) ? to_ticks(__builtin_bit_cast(float, waits), a.bounds.narrow) : 0ull);
    c0 = R - c0 > kSeqChunk ? c0 + kSeqChunk : R;
    __syncthreads();
  }
}

// kOne: every set's window is one request.  kFits: narrow_queue.
template <bool kScore, int S, bool kOne, bool kFits>
__global__ __launch_bounds__(kSeqThreads, S <= 2 ? 8 : (kScore ? 4 : 5)) void sweep_seq_kernel(const SweepWindowArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float4* rows = reinterpret_cast<float4*>(smem);
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ SeqChunks chunks;

  const uint32_t tid = threadIdx.x;
  const uint32_t lane = tid & 63u;
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6));
  const uint32_t n_waves = blockDim.x >> 6;  // candidates of a block
  const uint32_t blocks_per_set = (a.n_cand + n_waves - 1u) / n_waves;
  const uint32_t set = blockIdx.x / blocks_per_set;
  const uint32_t c = (blockIdx.x - set * blocks_per_set) * n_waves + wave;
  const bool mine_c = c < a.n_cand;  // a block's last wavefronts may have no candidate: they only prepare
  const SweepWindowSet rs = resolve_set(a.sets[set]);
  if (tid < a.n_slo) cls[tid] = ClassRow{a.d_ttft[tid], a.d_tbt[tid], a.i_ttft[tid], a.i_tbt[tid]};
  load_seq_rows(rows, a.tab, a.cells, a.mp, rs.window);

  const size_t base = (size_t)c * a.i_pad;
  const uint32_t n = mine_c ? min(a.n_inst[c], a.i_pad) : 0u;
  uint32_t tp[S], B[S];
  int32_t occ[S];
  uint64_t q[S];
  bool narrow = kFits;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    tp[s] = 0u; B[s] = 1u; occ[s] = 0; q[s] = 0ull;
    if (j < n) { tp[s] = a.tp_idx[base + j]; B[s] = a.max_batch[base + j]; occ[s] = a.occ[base + j]; q[s] = a.q_ticks[base + j]; }
    narrow = narrow && NarrowSequence<S>::fits(a.mp, tp[s], B[s], occ[s], q[s], rs.n_req);
  }
  narrow = __syncthreads_and(narrow) != 0;  // (the rows are complete as well)

  unsigned long long served[S], bad = 0ull;
  float inv_tbt_first[S];
  uint32_t sat = 0;                    // uniform
  unsigned long long wait_sum = 0ull;  // queue waits of the admitted requests, in ticks; uniform
#pragma unroll
  for (int s = 0; s < S; ++s) served[s] = 0ull;
  auto run = [&](auto& sq) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < S; ++s) sq.load(s, (uint32_t)s * 64u + lane < n, a.mp, a.cells, tp[s], B[s], occ[s], q[s]);
    sq.begin(rows, a.mp);
#pragma unroll
    for (int s = 0; s < S; ++s) inv_tbt_first[s] = kScore ? (sq.past[s] == INFINITY ? 0.0f : 1.0f / sq.rec[s].tbt) : 0.0f;
    walk_windows<kScore, S, kOne>(a, rs, sq, rows, cls, chunks, lane, wave, n_waves, served, sat, wait_sum);
  };
  if (kFits && narrow) {
    NarrowSequence<S> sq;
    run(sq);
  } else {
    Sequence<S, kFits> sq;
    run(sq);
    bad = sq.bad;
  }

  // results of this (set, candidate): lane 0 writes them
  if (bad != 0ull && rs.n_req != 0u) raise_status(a.status, 2u);  // (a lane without an instance is never bad)
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
struct SeqOutputs {
  int idx, slack, ttft, tbt, e2e;  // bit patterns; request c0 + lane in this lane
};

// A chunk of requests in LDS, and what of it stays in registers: its valid requests, the time behind each.
struct AssignChunk {
  float4 u[kSeqChunk + 1], w[kSeqChunk + 1];  // RequestSide; the last is read ahead and never used
};

template <bool kLat>
__device__ __forceinline__ void store_outputs(const AssignArgs& a, uint32_t c0, uint32_t lane, unsigned long long live,
                                              const SeqOutputs& o) {
  const uint32_t r = c0 + lane;
  if (r >= a.n_req) return;
  const float slack = __builtin_bit_cast(float, o.slack), nanv = __builtin_nanf("");
  const bool given = in_mask(live) && slack > -INFINITY;  // a class out of range, or no instance
  if (a.chosen) a.chosen[r] = given ? o.idx : -1;
  if (a.slack) a.slack[r] = given ? slack : -INFINITY;
  if (kLat) {
    if (a.ttft) a.ttft[r] = given ? __builtin_bit_cast(float, o.ttft) : nanv;
    if (a.tbt) a.tbt[r] = given ? __builtin_bit_cast(float, o.tbt) : nanv;
    if (a.e2e) a.e2e[r] = given ? __builtin_bit_cast(float, o.e2e) : nanv;
  }
}

// Requests r0 .. r0 + 63 as they come from memory, with the arrivals of them and of those behind them.
struct AssignRaw {
  RequestRaw rq;
  uint32_t own, behind;
};
__device__ __forceinline__ AssignRaw fetch_assign(const AssignArgs& a, uint32_t c0, uint32_t lane) {
  const uint32_t r = c0 + lane;
  AssignRaw x{{0u, 0u, kNoRequest}, 0u, 0u};
  if (r < a.n_req) { x.rq.pl = a.prompt_len[r]; x.rq.ol = a.out_len[r]; x.rq.k = a.slo_class[r]; x.own = a.arrival_ticks[r]; }
  x.behind = x.own;
  if (r < a.n_req && a.n_req - r > 1u) x.behind = a.arrival_ticks[r + 1u];
  return x;
}

// The largest slack over the wavefront, uniform, and in the two wait states that a DPP operand needs behind the
// instruction that wrote it (twelve of them): the prefill in ticks of a request admitted by this lane, and the
// wait past the batch cap, (ov / B) * s_bar * tbt, of its instance if it does.
__device__ __forceinline__ float max_beside(float slack, float pre, float tbt, uint32_t load, uint32_t B, float invB,
                                            float s_bar, uint32_t& ticks, float& past) {
  float m, ov;
  asm("v_mul_f32 %[t], %[k], %[pre]\n\t"
      "v_mul_f32 %[w], %[sb], %[tbt]\n\t"
      "v_max_f32_dpp %[m], %[s], %[s] quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_rndne_f32 %[t], %[t]\n\t"
      "v_sub_u32 %[o], %[n], %[b] clamp\n\t"
      "v_max_f32_dpp %[m], %[m], %[m] quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_cvt_u32_f32 %[t], %[t]\n\t"
      "v_cvt_f32_u32 %[o], %[o]\n\t"
      "v_max_f32_dpp %[m], %[m], %[m] row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_mul_f32 %[o], %[o], %[i]\n\t"
      "s_nop 0\n\t"
      "v_max_f32_dpp %[m], %[m], %[m] row_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_mul_f32 %[w], %[o], %[w]\n\t"
      "s_nop 0\n\t"
      "v_max_f32_dpp %[m], %[m], %[m] row_bcast:15 row_mask:0xa bank_mask:0xf\n\t"
      "s_nop 1\n\t"
      "v_max_f32_dpp %[m], %[m], %[m] row_bcast:31 row_mask:0xc bank_mask:0xf"
      : [m] "=&v"(m), [t] "=&v"(ticks), [w] "=&v"(past), [o] "=&v"(ov)
      : [s] "v"(slack), [pre] "v"(pre), [tbt] "v"(tbt), [n] "v"(load), [b] "v"(B), [i] "v"(invB), [sb] "s"(s_bar),
        [k] "s"(1048576.0f));
  return lane_value(m, 63);
}

// A chunk of requests one by one, one slot per lane, while nothing completes: a chain of some sixty instructions
// without a branch.  What bounds it is the length of that chain: alone on its SIMD a wavefront issues an
// instruction every 4 cycles, whether it depends on the one before or not; a taken branch costs 20, a scalar
// instruction behind the vector one that wrote its operand 16 to 24, a table row from LDS some 100.  16,384 requests,
// 64 slots: 5.95 -> 4.94 ms with NarrowSequence (as it still is over more slots: 120: 0.54 -> 0.29 us per request) ->
// 2.72 with the chain -> 2.35 (0.143 us per request) with two requests a trip and the waits filled.  What an instance will be once it has admitted one more request is worked out ahead, so
// that the admission is a select; its row of the tables arrives while the next request is scored.
template <bool kLat, bool kPenalty>
__device__ __forceinline__ void assign_chain(const AssignArgs& a, NarrowSequence<1>& sq, const float4* rows,
                                             const AssignChunk& chunk, uint32_t gap, uint32_t len, SeqOutputs& o) {
  uint32_t w = sq.batch(0, sq.arr[0] + 1u, a.mp);
  float4 next = sq.row(0, w, rows);
  // request i, and the one that is `ahead` read meanwhile
  auto step = [&](uint32_t i, const RequestSide& q, uint32_t ahead) __attribute__((always_inline)) {
    const float wait = fmaf((float)sq.q[0], 0x1p-20f, sq.past[0]);
    const Deadlines d{q.u.y, q.u.z, q.w.z, q.w.x, q.w.y, q.w.w};
    const Margins g = score_triple(sq.rec[0].a, sq.rec[0].p, sq.rec[0].tbt, wait, q.u.x, q.u.w, d);
    const float next_tbt = kPenalty ? sq.penalised(0, next.z, w, a.mp) : next.z;
    const uint32_t load = sq.arr[0] + 1u;
    uint32_t ticks;
    float past;
    const float best = max_beside(g.slack, g.pre, next_tbt, load, sq.B[0], sq.invB[0], a.mp.s_bar, ticks, past);
    const unsigned long long held = lane_mask(g.slack == best);
    // a scalar instruction waits some 16 cycles for a mask that a vector one wrote: what does not depend on it
    // goes in between
    __builtin_amdgcn_sched_barrier(0);
    const RequestSide r{chunk.u[ahead], chunk.w[ahead]};
    const uint32_t passed = (uint32_t)__builtin_amdgcn_readlane((int)gap, (int)i);
    o.slack = with_lane(o.slack, (int)i, best);
    __builtin_amdgcn_sched_barrier(0);
    const uint32_t j = (uint32_t)__builtin_ctzll(held);  // (some lane holds it)
    const unsigned long long takes = __builtin_bit_cast(int, best) >= 0 ? 1ull << j : 0ull;
    if (kLat) {
      o.ttft = with_lane(o.ttft, (int)i, lane_value(g.ttft, (int)j));
      o.tbt = with_lane(o.tbt, (int)i, lane_value(sq.rec[0].tbt, (int)j));
      o.e2e = with_lane(o.e2e, (int)i, lane_value(g.e2e, (int)j));
    }
    o.idx = with_lane(o.idx, (int)i, (int)j);
    const bool me = in_mask(takes);
    sq.arr[0] = me ? load : sq.arr[0];
    w = sq.batch(0, sq.arr[0] + 1u, a.mp);
    const float4 row = sq.row(0, w, rows);
    __builtin_amdgcn_sched_barrier(0);  // (the read first: the next request's arithmetic hides it)
    sq.q[0] = __builtin_elementwise_sub_sat(sq.q[0] + (me ? ticks : 0u), passed);
    sq.rec[0].a = me ? next.x : sq.rec[0].a;
    sq.rec[0].p = me ? next.y : sq.rec[0].p;
    sq.rec[0].tbt = me ? next_tbt : sq.rec[0].tbt;
    sq.past[0] = me ? past : sq.past[0];
    next = row;
    return r;
  };
  RequestSide q{chunk.u[0], chunk.w[0]};
  uint32_t i = 0;
  for (; i + 2u <= len; i += 2u) {  // two a trip: what the next one reads needs no moves
    const RequestSide second = step(i, q, i + 1u);
    q = step(i + 1u, second, i + 2u);
  }
  if (i < len) step(i, q, i + 1u);
}

// Windows of `window` requests (kOne: of one), any state.  `tbt_min`: least entry of the per-token latency table.
template <bool kLat, int S, bool kOne, class Seq>
__device__ __forceinline__ unsigned long long assign_windows(const AssignArgs& a, uint32_t window, Seq& sq, const float4* rows,
                                                             const ClassRow* cls, AssignChunk& chunk, float tbt_min, uint32_t lane) {
  constexpr bool kChain = kOne && S == 1 && Seq::kNarrow;
  const uint32_t R = a.n_req;
  unsigned long long sat = 0ull;
  AssignRaw raw = fetch_assign(a, 0u, lane);
  uint32_t in_window = 0, delta = 0;
  for (uint32_t c0 = 0; c0 < R; c0 = R - c0 > kSeqChunk ? c0 + kSeqChunk : R) {
    const uint32_t len = min(R - c0, kSeqChunk);
    // one wavefront: its LDS operations stay in order, no barrier between the writes and the reads
    const unsigned long long live = lane_mask(raw.rq.k < a.n_slo);
    const RequestSide mine = request_side(raw.rq, a.n_slo, cls, a.status);
    chunk.u[lane] = mine.u;
    chunk.w[lane] = mine.w;
    const uint32_t gap = raw.behind - raw.own;  // (none behind the last request)
    if (R - c0 > kSeqChunk) raw = fetch_assign(a, c0 + kSeqChunk, lane);
    SeqOutputs o{0, 0, 0, 0, 0};
    const uint32_t at_most = kOne ? (uint32_t)__builtin_amdgcn_readfirstlane((int)~min_lanes<64>(~gap)) : 0u;
    bool done = false;
    if constexpr (kChain) {
      // nothing completes in this chunk: no gap in it reaches what the shortest service time allows with as
      // many requests running as there may be by its end
      const uint32_t run = min(sq.B[0], sq.arr[0] + kSeqChunk);
      const uint32_t most = ~min_lanes<64>(~run);
      if (at_most < (uint32_t)__builtin_amdgcn_readfirstlane((int)row_safe_ticks(a.mp.s_bar, tbt_min, most, 1u))) {
        if (a.mp.pen_kappa != 0.0f) assign_chain<kLat, true>(a, sq, rows, chunk, gap, len, o);
        else assign_chain<kLat, false>(a, sq, rows, chunk, gap, len, o);
        done = true;
      } else {
        sq.begin(rows, a.mp);
      }
    }
    for (uint32_t i = done ? len : 0u; i < len;) {
      if (kOne || in_window == 0u) sq.open_window();
      const uint32_t stop = kOne ? i + 1u : min(len, i + (window - in_window));  // of the window's requests in this chunk
      in_window += stop - i;
      do {
        const float best = score_slots<S>(RequestSide{chunk.u[i], chunk.w[i]}, sq.rec, sq.pre, sq.slack, sq.ttft, sq.e2e);
        const uint32_t j = holder_of<S>(sq.slack, best), l = j & 63u;
        o.idx = with_lane(o.idx, (int)i, (int)j);
        o.slack = with_lane(o.slack, (int)i, best);
#pragma unroll
        for (int s = 0; s < S; ++s)
          if (j >> 6 == (uint32_t)s) {
            rare_path();
            if (kLat) {  // what is reported about the chosen instance comes from the lane that holds it
              o.ttft = with_lane(o.ttft, (int)i, lane_value(sq.ttft[s], (int)l));
              o.tbt = with_lane(o.tbt, (int)i, lane_value(sq.rec[s].tbt, (int)l));
              o.e2e = with_lane(o.e2e, (int)i, lane_value(sq.e2e[s], (int)l));
            }
            // admitted: it loads the instance; a blocked request does not
            if (__builtin_bit_cast(int, best) >= 0) sq.template admit<kOne>(s, l, rows, a.mp);
          }
        delta += (uint32_t)__builtin_amdgcn_readlane((int)gap, (int)i);
      } while (++i < stop && !kOne);
      const bool last = c0 + stop == R;
      if (kOne || in_window == window || last) {
        const uint32_t passed = last ? 0u : delta;
        sq.template close_window<kOne>(passed, kOne ? at_most : passed, last, rows, a.mp);
        in_window = 0u;
        delta = 0u;
      }
    }
    sat += (unsigned long long)__popcll(lane_mask(lane < len && o.slack >= 0));
    store_outputs<kLat>(a, c0, lane, live, o);
  }
  return sat;
}

// kFits: narrow_queue.
template <bool kLat, int S, bool kFits>
__global__ __launch_bounds__(64) void assign_seq_kernel(const AssignArgs a, uint32_t window) {
  extern __shared__ __align__(16) unsigned char smem[];
  float4* rows = reinterpret_cast<float4*>(smem);
  __shared__ ClassRow cls[kMaxSlo];
  __shared__ AssignChunk chunk;
  const uint32_t lane = threadIdx.x;
  if (lane < a.n_slo) cls[lane] = ClassRow{a.d_ttft[lane], a.d_tbt[lane], a.i_ttft[lane], a.i_tbt[lane]};
  load_seq_rows(rows, a.tab, a.cells, a.mp, window);
  __syncthreads();
  float tbt_min = INFINITY;  // over the rows that are read
  for (uint32_t i = lane; i < a.cells; i += 64u)
    if (i % (a.mp.b_cap + 1u) != 0u) tbt_min = fminf(tbt_min, rows[i].z);
  tbt_min = -max_lanes<64>(-tbt_min);

  const PlacementRow row = select_row(a);
  const uint32_t n = row.n;
  uint32_t tp[S], B[S];
  int32_t occ[S];
  uint64_t q[S];
  bool narrow = kFits;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    const uint32_t j = (uint32_t)s * 64u + lane;
    tp[s] = 0u; B[s] = 1u; occ[s] = 0; q[s] = 0ull;
    if (j < n) { tp[s] = row.tp_idx[j]; B[s] = row.max_batch[j]; occ[s] = row.occ[j]; q[s] = row.q_ticks[j]; }
    narrow = narrow && NarrowSequence<S>::fits(a.mp, tp[s], B[s], occ[s], q[s], a.n_req);
  }
  narrow = lane_mask(!narrow) == 0ull;
  unsigned long long sat = 0ull;  // uniform
  auto run = [&](auto& sq) __attribute__((always_inline)) {
#pragma unroll
    for (int s = 0; s < S; ++s) sq.load(s, (uint32_t)s * 64u + lane < n, a.mp, a.cells, tp[s], B[s], occ[s], q[s]);
    sq.begin(rows, a.mp);
    if (window == 1u) sat = assign_windows<kLat, S, true>(a, 1u, sq, rows, cls, chunk, tbt_min, lane);
    else sat = assign_windows<kLat, S, false>(a, window, sq, rows, cls, chunk, tbt_min, lane);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const uint32_t j = (uint32_t)s * 64u + lane;
      if (j < n) { row.occ[j] = sq.occupancy(s); row.q_ticks[j] = sq.queue(s); }
    }
  };
  if (kFits && narrow) {
    NarrowSequence<S> sq;
    run(sq);
  } else {
    Sequence<S, kFits> sq;
    run(sq);
    if (sq.bad != 0ull) raise_status(a.status, 2u);
  }
  if (lane == 0u && a.n_satisfied) *a.n_satisfied = sat;
}

}  // namespace maaso
