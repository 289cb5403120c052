// Windows of requests laid out by class and prompt length, and what a placement admits of such a window.
//
// Within a window every request meets the same instance state, and of a request only its class and its prompt
// length decide - but for roundings - which instance takes it: the end-to-end margin lies between the two others.
// So a window's requests are dealt into batches of 64 of one class and of neighbouring lengths, once for all
// candidates, and a wavefront settles 64 batches at a time, a batch per lane, from the shortest and the longest
// prompt in it: nobody admits any of it, or one instance takes all of it, or it is left open and scored request
// by request.  What is left to do for a settled batch is to add up its prefills.
//
// Settled batches among those scored: capacity-aware config 4 (eight classes, windows of 4096, 2.7 instances that
// count) 94 %, Alg. 2's growth chains (two classes, windows of 256) 99 %.
#pragma once

#include "live_slots.hpp"
#include "sweep_window_kernels.hpp"

#pragma clang fp contract(off)

namespace maaso {

constexpr uint32_t kSegment = 4096;  // requests of a window that are laid out together
constexpr uint32_t kGroup = 256;     // requests that a wavefront reads at once, four per lane

// Batches of a segment of `requests` requests of n_slo classes, in whole groups: every class fills its last one up.
constexpr uint32_t segment_batches(uint32_t requests, uint32_t n_slo, uint32_t batch) {
  const uint32_t in_group = kGroup / batch;
  return (requests / batch + n_slo + in_group - 1u) / in_group * in_group;
}

// One batch: shortest and longest prompt, longest output, class and requests (0: an empty batch).
struct __align__(16) Batch {
  float lo, hi, out;
  uint32_t kn;
  __device__ __forceinline__ uint32_t k() const { return kn >> 16; }
  __device__ __forceinline__ uint32_t n() const { return kn & 0xffffu; }
};

// The load that `v` comes from has ended behind this.
__device__ __forceinline__ void arrived(f32x4& v) { asm volatile("" : "+v"(v)); }

__device__ __forceinline__ Batch batch_of(const f32x4& v) { return Batch{v.x, v.y, v.z, __float_as_uint(v.w)}; }

// A request set laid out: window w has `batches` batches from w * batches on, batch b of `size` requests its own from
// size * b on.
struct OrderedSet {
  uint32_t segments;  // of a window
  uint32_t batches;   // of a window, whole groups
  uint32_t size_log2;
  float* len;         // prompt lengths, zero behind a batch's last request
  float* out;         // output lengths
  Batch* batch;
  uint32_t* gap;      // [windows] ticks until the next window opens
};

struct OrderArgs {
  uint32_t n_slo;
  uint32_t* status;
  uint32_t n_sets;
  uint32_t first[kMaxSweepSets];  // first block of a set; a block per segment of a window
  SweepWindowSet sets[kMaxSweepSets];
  OrderedSet to[kMaxSweepSets];
};
constexpr uint32_t kOrderPer = 4;  // requests per thread
constexpr size_t order_lds(uint32_t segment, uint32_t n_slo, uint32_t batch) {
  return ((size_t)n_slo * kLenBins + 2u * kMaxSlo + 2u * batch * segment_batches(segment, n_slo, batch)) * sizeof(uint32_t);
}

// Counting sort of a segment in LDS, eight bins per octave of the length: within a bin the order is any, and no
// result depends on it.  What bounds it: latency, a few trips to memory and five barriers.
__global__ __launch_bounds__(1024) void order_requests_kernel(const OrderArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  uint32_t* bins = reinterpret_cast<uint32_t*>(smem);  // [n_slo][kLenBins]
  uint32_t* total = bins + a.n_slo * kLenBins;         // [kMaxSlo] requests of a class
  uint32_t* base = total + kMaxSlo;                    // [kMaxSlo] its first place
  float* len = reinterpret_cast<float*>(base + kMaxSlo);
  uint32_t set = 0;
  while (set + 1u < a.n_sets && blockIdx.x >= a.first[set + 1u]) ++set;
  const SweepWindowSet rs = resolve_set(a.sets[set]);
  const OrderedSet to = a.to[set];
  const uint32_t local = blockIdx.x - a.first[set];
  const uint32_t w = local / to.segments, seg = local - w * to.segments;
  if ((uint64_t)w * rs.window >= rs.n_req) return;  // (a side of a split may be shorter than the whole)
  const uint32_t s0 = w * rs.window;
  const uint32_t e0 = rs.n_req - s0 > rs.window ? s0 + rs.window : rs.n_req;
  const uint32_t skip = seg * kSegment;
  const uint32_t n = e0 - s0 > skip ? min(e0 - s0 - skip, kSegment) : 0u;
  const uint32_t r0 = s0 + skip;
  const uint32_t size = 1u << to.size_log2;
  const uint32_t places = (to.batches / to.segments) << to.size_log2;
  float* out = len + places;

  const uint32_t tid = threadIdx.x, T = blockDim.x, lane = tid & 63u, wave = tid >> 6, waves = T >> 6;
  if (tid == 0u && seg == 0u) to.gap[w] = e0 < rs.n_req ? rs.arrival_ticks[e0] - rs.arrival_ticks[s0] : 0u;
  uint32_t pl[kOrderPer], ol[kOrderPer], k[kOrderPer];
#pragma unroll
  for (uint32_t u = 0; u < kOrderPer; ++u) {
    const uint32_t i = u * T + tid;
    pl[u] = ol[u] = 0u;
    k[u] = kNoRequest;
    if (i < n) { pl[u] = rs.prompt_len[r0 + i]; ol[u] = rs.out_len[r0 + i]; k[u] = rs.slo_class[r0 + i]; }
  }
  for (uint32_t i = tid; i < a.n_slo * kLenBins; i += T) bins[i] = 0u;
  for (uint32_t i = tid; i < places; i += T) { len[i] = 0.0f; out[i] = 0.0f; }
  __syncthreads();
  uint32_t bin[kOrderPer], at[kOrderPer];
#pragma unroll
  for (uint32_t u = 0; u < kOrderPer; ++u) {
    if (k[u] >= a.n_slo) {  // a class out of range is served by nobody
      if (k[u] != kNoRequest) raise_status(a.status, 1u);
      k[u] = kNoRequest;
      continue;
    }
    bin[u] = k[u] * kLenBins + length_bin((float)pl[u]);
    at[u] = atomicAdd(&bins[bin[u]], 1u);
  }
  __syncthreads();
  for (uint32_t c = wave; c < a.n_slo; c += waves) {  // exclusive prefix over a class's bins, four per lane
    static_assert(kLenBins == 256u, "four bins per lane");
    uint4* mine = reinterpret_cast<uint4*>(bins + c * kLenBins) + lane;
    const uint4 v = *mine;
    const uint32_t sum = v.x + v.y + v.z + v.w;
    uint32_t inc = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t o = __shfl_up(inc, d);
      if (lane >= (uint32_t)d) inc += o;
    }
    const uint32_t b = inc - sum;
    *mine = make_uint4(b, b + v.x, b + v.x + v.y, b + v.x + v.y + v.z);
    if (lane == 63u) total[c] = inc;
  }
  __syncthreads();
  if (tid < a.n_slo) {
    uint32_t b = 0;
    for (uint32_t c = 0; c < tid; ++c) b += (total[c] + size - 1u) & ~(size - 1u);
    base[tid] = b;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t u = 0; u < kOrderPer; ++u) {
    if (k[u] == kNoRequest) continue;
    const uint32_t p = base[k[u]] + bins[bin[u]] + at[u];
    len[p] = (float)pl[u];
    out[p] = (float)ol[u];
  }
  __syncthreads();
  const size_t p0 = ((size_t)w * to.batches << to.size_log2) + (size_t)seg * places;
  for (uint32_t p = tid; p < places; p += T) {  // (whole wavefronts: groups of 256)
    const uint32_t first = p & ~(size - 1u);
    uint32_t c = 0;  // the last class that begins here or before (an empty class begins where the next does)
    for (uint32_t i = 1; i < a.n_slo; ++i) c = base[i] <= first ? i : c;
    const uint32_t cnt = total[c] > first - base[c] ? min(total[c] - (first - base[c]), size) : 0u;
    const float L = len[p];
    const uint32_t bits = __float_as_uint(L);  // (not negative: in order as they are)
    const bool own = p - first < cnt;
    const float So = out[p];
    uint32_t lo = min_lanes<16>(own ? bits : 0xffffffffu), hi = min_lanes<16>(own ? ~bits : 0xffffffffu);
    uint32_t most = min_lanes<16>(own ? ~__float_as_uint(So) : 0xffffffffu);
    for (uint32_t d = 16; d < size; d <<= 1) {
      lo = min(lo, (uint32_t)__shfl_xor((int)lo, (int)d));
      hi = min(hi, (uint32_t)__shfl_xor((int)hi, (int)d));
      most = min(most, (uint32_t)__shfl_xor((int)most, (int)d));
    }
    to.len[p0 + p] = L;
    to.out[p0 + p] = So;
    if (p == first)
      to.batch[(p0 + p) >> to.size_log2] = cnt ? Batch{__uint_as_float(lo), __uint_as_float(~hi), __uint_as_float(~most), c << 16 | cnt}
                                               : Batch{0.0f, 0.0f, 0.0f, 0u};
  }
}

// Prefill ticks of every batch on every row of the profile tables, where windows are long and requests many (sweep_sums_batches):
// ticks[row * n_batches + b].  A batch whose longest prompt takes eight seconds and more on
// a row has no sum here, and none is looked up.
struct TicksArgs {
  const float* tab;
  uint32_t cells;
  const float* len;
  const Batch* batch;
  uint32_t n_batches;  // of all windows, whole groups
  uint32_t* ticks;
};

// How the NW wavefronts that share a window take its batches of 2^kLog2 requests: groups in turn, 64 batches a pass.
template <int NW, int kLog2>
struct Dealt {
  static constexpr uint32_t kIn = kGroup >> kLog2;  // batches of a group
  static constexpr uint32_t kPass = 64u / kIn;      // groups of a pass
  uint32_t wave, lane;

  __device__ __forceinline__ uint32_t group(uint32_t pass, uint32_t i) const { return wave + (uint32_t)NW * (kPass * pass + i); }
  __device__ __forceinline__ uint32_t batch(uint32_t pass, uint32_t l) const { return kIn * group(pass, l / kIn) + l % kIn; }
  __device__ __forceinline__ bool any(const OrderedSet& os, uint32_t pass) const { return kIn * group(pass, 0u) < os.batches; }
  // (a lane beyond the window's batches reads the last one: see holds)
  __device__ __forceinline__ f32x4 read_batch(const OrderedSet& os, uint32_t w, uint32_t pass) const {
    return reinterpret_cast<const f32x4*>(os.batch)[(size_t)w * os.batches + min(batch(pass, lane), os.batches - 1u)];
  }
  __device__ __forceinline__ bool holds(const OrderedSet& os, uint32_t pass) const { return batch(pass, lane) < os.batches; }
  __device__ __forceinline__ f32x4 read_lengths(const OrderedSet& os, uint32_t w, uint32_t pass, uint32_t i) const {
    const uint32_t g = min(group(pass, i), os.batches / kIn - 1u);
    return reinterpret_cast<const f32x4*>(os.len + (((size_t)w * os.batches) << kLog2))[g * 64u + lane];
  }
};

// Prefills are added up as ticks of 2^-20 s: below 8 s the sum 8 + x has its last place there, so that one
// addition rounds x to ticks, to nearest even as rint does, and leaves them in the low bits.
constexpr float kTickBase = 8.0f;
__device__ __forceinline__ uint32_t tick_bits(float pre) { return __float_as_uint(pre + kTickBase); }

// A wavefront takes a group of four batches of 64, four requests per lane, through 64 rows.
__global__ __launch_bounds__(256) void batch_ticks_kernel(const TicksArgs a) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t g = blockIdx.x * 4u + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  if (4u * g >= a.n_batches) return;
  const f32x4 len = reinterpret_cast<const f32x4*>(a.len)[(size_t)g * 64u + lane];
  const uint32_t b = 4u * g + (lane >> 4), filler = 64u - a.batch[b].n();
  const uint32_t r0 = blockIdx.y * 64u, rows = min(64u, a.cells - r0);
  const uint32_t own = r0 + min(lane, rows - 1u);
  const float own_a = a.tab[own], own_p = a.tab[a.cells + own];
  uint32_t* to = a.ticks + (size_t)r0 * a.n_batches + b;
  for (uint32_t r = 0; r < rows; ++r, to += a.n_batches) {
    const float ra = lane_value(own_a, (int)r), rp = lane_value(own_p, (int)r);
    const uint32_t t = row_sum_u32(tick_bits(fmaf(rp, len.x, ra)) + tick_bits(fmaf(rp, len.y, ra)) +
                                   tick_bits(fmaf(rp, len.z, ra)) + tick_bits(fmaf(rp, len.w, ra)));
    // the places behind a batch's last request hold length 0: they counted with the prefill of none
    if ((lane & 15u) == 0u)
      *to = t - 64u * __float_as_uint(kTickBase) - filler * (tick_bits(ra) - __float_as_uint(kTickBase));
  }
}

// What each lane's batch comes to: kOpen, kNobody, or the instance that takes all of it.
constexpr uint32_t kOpen = 0xffffffffu, kNobody = 0xfffffffeu;

// A batch against one instance: its largest and its least slack over the batch, as far as they are known (see
// settle_batch), and the prefill of the longest prompt.  Under the shortest-queue rule (kSQ) its rank, or -1, if it serves
// any of the batch, and if it serves all of it.
struct BatchBounds {
  float up, low, longest;
};
template <bool kSQ>
__device__ __forceinline__ BatchBounds batch_bounds(const Batch& b, const ClassRow& c, float clear, const SlotRecord& r, float rank) {
  BatchBounds x;
  const float s2 = (c.Db - r.tbt) * c.iDb;
  x.longest = fmaf(r.p, b.hi, r.a);
  const float s1 = (c.Dt - (r.wait + x.longest)) * c.iDt;
  x.up = fminf((c.Dt - (r.wait + fmaf(r.p, b.lo, r.a))) * c.iDt, s2);
  x.low = fminf(s1 - clear, s2);
  if (kSQ) {
    x.up = x.up >= 0.0f ? rank : -1.0f;
    x.low = fminf(s1, s2) >= 0.0f ? rank : -1.0f;
  }
  return x;
}

// The bounds.  All operations are monotone, so an instance's largest slack over a batch is at most the lesser of its
// margins s1 (first token) and s2 (between tokens) at the shortest prompt, and the lesser of the two at the longest
// is its least, were it not for the end-to-end margin s3.  That one lies between them, f = Dt / De of the way from s2
// to s1, De = Dt + S Db, but as computed may come out below both.  With u = 2^-24, where both latencies are within
// their deadlines: s3 is within 5.2 u of its value (a rounding each in the two sums, whose quotient is at most 1, in
// the difference, the reciprocal and the product), s1 and s2 within 3.1 u each, so s3 >= s2 + f (s1 - s2) - 14.5 u as
// computed.  With c = 16 u / f (f of the batch's longest output) the least slack is not below min(s1 - c, s2), s1 at the longest
// prompt: for s1 <= s2 and for s1 >= s2 + c that is plain, between them f d - 14.5 u >= d - c for 0 <= d <= c.  On s2 that bound is exact:
// instances of one kind tie there, and the first takes the batch.
//
// An instance takes a batch if it serves the longest prompt, and so all, and its least slack is above every other's
// largest, or equal for those behind it: it is then the first with the largest largest slack.  Under the shortest-queue rule
// (kSQ) what is compared are ranks, of the instances that serve any of a batch, and of those that serve all of it.  `floor`:
// the largest of the least slacks, zero at least; an instance whose largest is below it is given nothing of the batch.
constexpr float kSlackSlip = 0x1p-20f;
template <int S, bool kSQ>
__device__ __forceinline__ uint32_t settle_batch(const Batch& b, bool holds, const ClassRow& c, float clear,
                                                 const SlotRecord (&rec)[S], const InstanceSet<S>& set, const float (&rank)[S],
                                                 float& floor) {
  float top = -INFINITY, second = -INFINITY, low = -INFINITY, pre = 0.0f;
  uint32_t holder = kOpen;
  floor = 0.0f;
#pragma unroll
  for (int s = 0; s < S; ++s) {
    for (unsigned long long todo = set.m[s]; todo != 0ull; todo &= todo - 1ull) {
      const int l = (int)__builtin_ctzll(todo);
      const BatchBounds x = batch_bounds<kSQ>(b, c, clear, rec[s].of_lane(l), kSQ ? lane_value(rank[s], l) : 0.0f);
      const bool first = x.up > top;
      holder = first ? (uint32_t)(s * 64 + l) : holder;
      low = first ? x.low : low;
      pre = first ? x.longest : pre;
      second = __builtin_amdgcn_fmed3f(top, second, x.up);
      top = max_no_nan(top, x.up);
      floor = max_no_nan(floor, x.low);
    }
  }
  const bool takes = (low >= 0.0f) & ((low > second) | (low == top)) & (pre < kTickBase);
  return !holds || b.kn == 0u || top < 0.0f ? kNobody : takes ? holder : kOpen;
}

// Ticks of four requests per lane where the lane's bit of `bits` (one per batch of the group) is set: all of them are of
// one batch.
template <int kLog2>
__device__ __forceinline__ uint32_t group_ticks(const f32x4& len, uint32_t bits, uint32_t lane, float a, float p) {
  const uint32_t t = tick_bits(fmaf(p, len.x, a)) + tick_bits(fmaf(p, len.y, a)) + tick_bits(fmaf(p, len.z, a)) +
                     tick_bits(fmaf(p, len.w, a)) - 4u * __float_as_uint(kTickBase);
  return t & (uint32_t)__builtin_amdgcn_sbfe((int)bits, lane >> (kLog2 - 2), 1u);
}

// A window's requests against the instances in `set` (not empty; a set that find_admissible found).  give(j, num, ticks),
// uniform: instance j takes num requests of `ticks` prefill in all.
// `batch`: the lane's of the first pass; `len`: its lengths in the wavefront's first kFirst groups, the only ones there are
// with kOnly.  A wavefront asks for both ahead of the evaluation of its instances.
// kTable: what batches add up to is in `ticks` (of this window; row_ticks entries on for every row of the tables), and row_of(j)
// says which row instance j is on.
template <int S, int NW, int kLog2, bool kSQ, int kFirst, bool kOnly, bool kTable, class Give, class RowOf>
__device__ __forceinline__ void score_window(const Dealt<NW, kLog2>& deal, const OrderedSet& os, uint32_t w, f32x4 batch,
                                             const f32x4 (&len)[kFirst ? kFirst : 1], const ClassRow* cls,
                                             const SlotRecord (&rec)[S], const int32_t (&occ)[S], const InstanceSet<S>& set,
                                             const uint32_t* ticks, uint32_t row_ticks, RowOf&& row_of, Give&& give) {
  static_assert(kFirst <= (int)Dealt<NW, kLog2>::kPass, "of the first pass");
  constexpr uint32_t kSize = 1u << kLog2, kIn = kGroup >> kLog2;
  const uint32_t lane = deal.lane;
  float rank[S];
#pragma unroll
  for (int s = 0; s < S; ++s) rank[s] = 0.0f;
  if (kSQ) queue_ranks<S>(occ, set, lane, rank);
  Batch b = batch_of(batch);
  for (uint32_t pass = 0;;) {
    const ClassRow row = cls[b.k()];
    const float clear = kSlackSlip * (fmaf(b.out, row.Db, row.Dt) * row.iDt);
    float floor;
    const uint32_t to = settle_batch<S, kSQ>(b, deal.holds(os, pass), row, clear, rec, set, rank, floor);
    for (unsigned long long todo = lane_mask(to < kNobody); todo != 0ull;) {
      const uint32_t j = (uint32_t)__builtin_amdgcn_readlane((int)to, (int)__builtin_ctzll(todo));
      const unsigned long long mask = lane_mask(to == j);
      todo &= ~mask;
      if constexpr (kTable) {
        const uint32_t t = in_mask(mask) ? ticks[(size_t)row_of(j) * row_ticks + deal.batch(pass, lane)] : 0u;
        uint32_t n = in_mask(mask) ? b.n() : 0u, sum = t & 0x3ffffffu;
        wave_sum_pair(n, sum);
        unsigned long long all = sum;
        if (lane_mask(t >> 26 != 0u) != 0ull) {
          rare_path();
          all += (unsigned long long)wave_sum_u32(t >> 26) << 26;
        }
        give(j, n, all);
        continue;
      }
      float a = lane_value(rec[0].a, (int)(j & 63u)), p = lane_value(rec[0].p, (int)(j & 63u));
#pragma unroll
      for (int s = 1; s < S; ++s)
        if (j >> 6 == (uint32_t)s) { a = lane_value(rec[s].a, (int)(j & 63u)); p = lane_value(rec[s].p, (int)(j & 63u)); }
      uint32_t acc = 0;  // a lane adds at most 64 requests of less than 2^23 ticks
      unsigned long long groups = mask;
      if (kFirst && pass == 0u) {
#pragma unroll
        for (int i = 0; i < kFirst; ++i) acc += group_ticks<kLog2>(len[i], (uint32_t)(mask >> (i * (int)kIn)), lane, a, p);
        groups = kOnly || kFirst == (int)Dealt<NW, kLog2>::kPass ? 0ull : mask >> (kFirst * kIn % 64u) << (kFirst * kIn % 64u);
      }
      if (!kOnly && groups != 0ull) {
        for (uint32_t d = 1; d < kIn; d <<= 1) groups |= groups >> d;  // bit kIn * i: some batch of the pass's group i
        groups &= kIn == 4u ? 0x1111111111111111ull : kIn == 8u ? 0x0101010101010101ull : 0x0001000100010001ull;
        if (kFirst && pass == 0u) groups = groups >> (kFirst * kIn % 64u) << (kFirst * kIn % 64u);
        f32x4 next = deal.read_lengths(os, w, pass, (uint32_t)__builtin_ctzll(groups) / kIn);
        while (groups != 0ull) {  // the next group is read ahead of its use
          const f32x4 v = next;
          const uint32_t bits = (uint32_t)(mask >> __builtin_ctzll(groups));
          groups &= groups - 1ull;
          if (groups != 0ull) next = deal.read_lengths(os, w, pass, (uint32_t)__builtin_ctzll(groups) / kIn);
          acc += group_ticks<kLog2>(v, bits, lane, a, p);
        }
      }
      // the places behind a batch's last request hold length 0: they counted with the prefill of none
      uint32_t n = in_mask(mask) ? b.n() : 0u, sum = acc & 0x3ffffffu;
      wave_sum_pair(n, sum);
      unsigned long long ticks = sum;
      if (lane_mask(acc >> 26 != 0u) != 0ull) {
        rare_path();
        ticks += (unsigned long long)wave_sum_u32(acc >> 26) << 26;
      }
      const uint32_t filler = kSize * (uint32_t)__popcll(mask) - n;
      give(j, n, ticks - (unsigned long long)filler * (tick_bits(a) - __float_as_uint(kTickBase)));
    }
    // the batches left open, a request per lane, V wavefronts' worth at a time and as many on their way
    unsigned long long open = lane_mask(to == kOpen);
    if (open != 0ull) {
      // with many instances, against those alone that may be given something of one of them
      InstanceSet<S> some = set;
      if (set.count() > 4u) {
#pragma unroll
        for (int s = 0; s < S; ++s)
          for (unsigned long long todo = set.m[s]; todo != 0ull; todo &= todo - 1ull) {
            const int l = (int)__builtin_ctzll(todo);
            const BatchBounds x = batch_bounds<kSQ>(b, row, clear, rec[s].of_lane(l), kSQ ? lane_value(rank[s], l) : 0.0f);
            if ((lane_mask(x.up >= floor) & open) == 0ull) some.m[s] &= ~(1ull << l);
          }
      }
      constexpr int V = kOnly ? 1 : 2;
      struct Asked {
        float L, out;
        uint32_t kn;
      };
      auto ask = [&](Asked (&q)[V]) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < V; ++v) {
          uint32_t at = 0, kn = 0;  // of this lane's batch
#pragma unroll
          for (uint32_t i = 0; i < 64u / kSize; ++i) {
            if (open == 0ull) continue;
            const int l = (int)__builtin_ctzll(open);
            open &= open - 1ull;
            const bool mine = lane >> kLog2 == i;
            at = mine ? deal.batch(pass, (uint32_t)l) : at;
            kn = mine ? (uint32_t)__builtin_amdgcn_readlane((int)b.kn, l) : kn;
          }
          const size_t r = (((size_t)w * os.batches + at) << kLog2) + (lane & (kSize - 1u));
          q[v] = Asked{os.len[r], os.out[r], kn};
        }
      };
      Asked next[V];
      ask(next);
      for (bool more = true; more;) {
        float L[V], So[V], best[V], pre[V];
        uint32_t kn[V], holder[V];
        Deadlines d[V];
#pragma unroll
        for (int v = 0; v < V; ++v) { L[v] = next[v].L; So[v] = next[v].out; kn[v] = next[v].kn; }
        more = open != 0ull;
        if (more) ask(next);
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const ClassRow c = cls[kn[v] >> 16];
          const float De = fmaf(So[v], c.Db, c.Dt);
          d[v] = Deadlines{c.Dt, c.Db, De, c.iDt, c.iDb, 1.0f / De};
          best[v] = -INFINITY;
          pre[v] = 0.0f;
          holder[v] = kNobody;
        }
#pragma unroll
        for (int s = 0; s < S; ++s)
          for (unsigned long long todo = some.m[s]; todo != 0ull; todo &= todo - 1ull) {
            const int l = (int)__builtin_ctzll(todo);
            const SlotRecord k = rec[s].of_lane(l);
            const float rk = kSQ ? lane_value(rank[s], l) : 0.0f;
#pragma unroll
            for (int v = 0; v < V; ++v) {
              const Margins g = score_triple(k.a, k.p, k.tbt, k.wait, L[v], So[v], d[v]);
              const float val = (kSQ && g.slack >= 0.0f) ? rk : g.slack;
              const bool better = val > best[v];
              holder[v] = better ? (uint32_t)(s * 64 + l) : holder[v];
              pre[v] = better ? g.pre : pre[v];
              best[v] = max_no_nan(best[v], val);
            }
          }
        uint32_t ticks[V];
        unsigned long long left[V];
#pragma unroll
        for (int v = 0; v < V; ++v) {
          ticks[v] = (uint32_t)rintf(pre[v] * 1048576.0f);
          left[v] = lane_mask(best[v] >= 0.0f) & lane_mask((lane & (kSize - 1u)) < (kn[v] & 0xffffu));
        }
        while ((left[0] | left[V - 1]) != 0ull) {
          const uint32_t j = left[0] != 0ull ? (uint32_t)__builtin_amdgcn_readlane((int)holder[0], (int)__builtin_ctzll(left[0]))
                                             : (uint32_t)__builtin_amdgcn_readlane((int)holder[V - 1], (int)__builtin_ctzll(left[V - 1]));
          uint32_t num = 0;
          unsigned long long sum = 0ull;
#pragma unroll
          for (int v = 0; v < V; ++v) {
            const unsigned long long mask = lane_mask(holder[v] == j) & left[v];
            left[v] &= ~mask;
            num += (uint32_t)__popcll(mask);
            sum += in_mask(mask) ? ticks[v] : 0u;
          }
          give(j, num, wave_sum_ticks(sum));
        }
      }
    }
    ++pass;
    if (kOnly || !deal.any(os, pass)) return;  // uniform
    f32x4 more = deal.read_batch(os, w, pass);
    arrived(more);  // here, so that the first pass waits for nothing that was asked for since
    b = batch_of(more);
  }
}

}  // namespace maaso
