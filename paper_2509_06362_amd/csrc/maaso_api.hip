// Host side of the C ABI declared in include/maaso.h: argument validation, the context, launch
// shapes.  Every step of the scoring path runs in the kernels of the headers below; nothing here
// computes on the CPU beyond table validation and the reciprocals of the class deadlines.
#include "../../include/maaso.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cfloat>
#include <cmath>
#include <cstring>
#include <new>
#include <type_traits>

#include "assign_kernels.hpp"
#include "assign_ordered_kernels.hpp"
#include "sweep_kernels.hpp"
#include "partition_kernels.hpp"
#include "probe_kernels.hpp"
#include "profile_fit_kernels.hpp"
#include "sweep_window_kernels.hpp"
#include "sweep_block_kernels.hpp"
#include "sweep_ordered_kernels.hpp"
#include "sweep_seq_kernels.hpp"
#include "window_kernels.hpp"

using namespace maaso;

static_assert(MAASO_MAX_SLO == kMaxSlo, "header and kernels disagree on the class limit");

constexpr uint32_t kMaxTimed = 256;
// The context's small device block, in 32-bit words: [0] status, [32..35] evaluated pairs of the last
// static sweep (all; those without a wait), [64..] the static distributor's admitted-count accumulators,
// then the static sweep's SweepTotals; from kCounterWord on its histogram, cursors and group offsets.
constexpr uint32_t kClassWord = 40;  // [kMaxSlo] requests of each class, between two launches of the static sweep
constexpr uint32_t kSatWord = 64;
static_assert(kClassWord + kMaxSlo <= kSatWord, "");
constexpr uint32_t kTotalsWord = kSatWord + (1u + kSatLines) * kSatStride * 2u;
constexpr uint32_t kCounterWord = kTotalsWord + (1u + kTotalsLines) * sizeof(SweepTotals) / 4u;
constexpr uint32_t kHistWords = kMaxSlo * kLenBins;
constexpr size_t kSmallBytes = ((size_t)kCounterWord + 3u * kHistWords + 64u) * 4u;
static_assert(kTotalsWord * 4u % alignof(SweepTotals) == 0u && sizeof(SweepTotals) == 128u, "");

// Workspace of maaso_placement_sweep_noalloc: device memory that exists from the moment the library
// is loaded, one copy per GPU, so that the call has nothing to allocate.  In host code the array's
// name is only a handle for hipGetSymbolAddress; kernels are given the address resolved per device.
constexpr int kMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[MAASO_NOALLOC_SCRATCH_BYTES];
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

struct maaso_ctx {
  int device;
  uint32_t n_tp, b_cap, cells, n_slo;
  float d_ttft[kMaxSlo], d_tbt[kMaxSlo], i_ttft[kMaxSlo], i_tbt[kMaxSlo];
  float tbt_min, tbt_max;  // least and largest entry of the per-token latency table
  float* tab;           // device: three tables back to back, then tp_degree [n_tp] as uint32
  bool has_degree;      // the profile came with GPUs-per-instance figures
  uint32_t* status;     // device status word
  void* scratch_ptr;    // this device's copy of the static scratch array
  void* ws;             // device workspace: sized at load, resized only by maaso_ctx_reserve
  size_t ws_bytes;
  uint32_t ws_allocations;  // how often the workspace has been allocated (load counts as one)
  size_t ws_low;        // bytes at its start that captured calls use, which may replay beside any later call
  // one call at a time: the host part of a call is exclusive, and a call on another stream than the
  // context's previous call is ordered behind it with an event
  std::atomic<int> in_call;
  hipEvent_t order_ev;
  hipStream_t last_stream;
  bool has_last;
  uint32_t sweep_q;      // 0 = automatic
  uint32_t sweep_group;  // 0 = automatic
  uint32_t sweep_blocks_per_queue;  // 0 = automatic
  unsigned long long* last_evaluated;  // device word written by the last sweep, or null
  bool counters_dirty;   // histogram, cursors or totals may be non-zero (a call failed between its launches)
  uint32_t window_blocks;  // 0 = automatic
  uint32_t spin_limit;     // polls of the inter-window barrier before a block gives up
  bool window_profile;     // the windowed distributor records where block 0 spends its cycles
  bool window_profiled;    // ... and the last windowed call did
  int n_cu;
  int cooperative;      // the device launches cooperative grids (all blocks resident, or refused)
  size_t lds_per_block;
  // optional timing of the dominant kernel of each call (HIP events on the call's stream)
  bool timing;
  uint32_t n_timed;
  hipEvent_t ev_start[kMaxTimed], ev_stop[kMaxTimed];
};

namespace {

struct DeviceGuard {
  int prev = -1;
  bool ok = true;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) { ok = false; (void)hipGetLastError(); return; }
    if (prev != dev && hipSetDevice(dev) != hipSuccess) { ok = false; (void)hipGetLastError(); }
  }
  ~DeviceGuard() {
    int cur = -1;
    if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
  }
};

inline bool hip_ok(hipError_t e) {
  if (e == hipSuccess) return true;
  (void)hipGetLastError();
  return false;
}

// Event pair around the dominant kernel of a call, when timing is on and slots are left.
struct TimedRegion {
  maaso_ctx* ctx;
  hipStream_t s;
  bool on;
  TimedRegion(maaso_ctx* c, hipStream_t st) : ctx(c), s(st), on(c->timing && c->n_timed < kMaxTimed) {
    if (on) on = hipEventRecord(ctx->ev_start[ctx->n_timed], s) == hipSuccess;
  }
  ~TimedRegion() {
    if (on && hipEventRecord(ctx->ev_stop[ctx->n_timed], s) == hipSuccess) ctx->n_timed += 1;
  }
};

// Compute calls never allocate: a call whose shape needs more than the context holds is refused.
int need_workspace(const maaso_ctx* ctx, size_t bytes) {
  return bytes <= ctx->ws_bytes ? MAASO_OK : MAASO_E_WORKSPACE;
}

bool is_captured(hipStream_t s) {
  if (s == nullptr) return false;  // (the null stream cannot be)
  hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
  return hip_ok(hipStreamIsCapturing(s, &status)) && status != hipStreamCaptureStatusNone;
}

// Calls that are charged with no workspace, the windowed sweep and the scores, lay requests out at its end, and keep out of what
// charged calls that were captured use at its start: these may replay beside any later call.  Others are ordered with them and leave
// all of it.  (It is asked only where that much is not kept already.)
void use_workspace(maaso_ctx* ctx, size_t bytes, hipStream_t s) {
  if (bytes > ctx->ws_low && is_captured(s)) ctx->ws_low = bytes;
}

// Set-up only (load, maaso_ctx_reserve): (re)allocates the workspace when it is too small.
int alloc_workspace(maaso_ctx* ctx, size_t bytes) {
  if (bytes <= ctx->ws_bytes) return MAASO_OK;
  if (ctx->ws) {
    if (!hip_ok(hipDeviceSynchronize())) return MAASO_E_HIP;
    (void)hipFree(ctx->ws);
    ctx->ws = nullptr;
    ctx->ws_bytes = ctx->ws_low = 0;
  }
  const size_t want = (bytes + (size_t(1) << 20) - 1) & ~((size_t(1) << 20) - 1);
  if (!hip_ok(hipMalloc(&ctx->ws, want))) { ctx->ws = nullptr; return MAASO_E_NOMEM; }
  ctx->ws_bytes = want;
  ctx->ws_allocations += 1;
  return MAASO_OK;
}

// Exclusive use of a context by one call, and stream order between consecutive calls.  The context's
// workspace, class counters and accumulators are shared by all its calls; calls issued on one stream
// are ordered by the stream, and a call issued on another stream than the previous one is made to
// wait for it: an event is recorded on the previous stream at that moment (it covers everything
// issued there so far) and the new stream waits for it - no host synchronisation.  Should the
// previous stream no longer exist, the device is synchronised instead.
struct CallGuard {
  maaso_ctx* ctx;
  int rc;
  CallGuard(maaso_ctx* c, hipStream_t s) : ctx(c), rc(MAASO_OK) {
    int idle = 0;
    if (!ctx->in_call.compare_exchange_strong(idle, 1, std::memory_order_acquire)) {
      ctx = nullptr;
      rc = MAASO_E_BUSY;
      return;
    }
    if (ctx->has_last && ctx->last_stream != s) {
      const bool ordered = hipEventRecord(ctx->order_ev, ctx->last_stream) == hipSuccess &&
                           hipStreamWaitEvent(s, ctx->order_ev, 0) == hipSuccess;
      if (!ordered) {
        (void)hipGetLastError();
        if (!hip_ok(hipDeviceSynchronize())) rc = MAASO_E_HIP;
      }
    }
    ctx->last_stream = s;
    ctx->has_last = true;
  }
  ~CallGuard() {
    if (ctx) ctx->in_call.store(0, std::memory_order_release);
  }
  CallGuard(const CallGuard&) = delete;
  CallGuard& operator=(const CallGuard&) = delete;
};

int check_common(const maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                 const maaso_params* prm) {
  if (!ctx || !pl || !rq || !prm) return MAASO_E_INVALID_ARG;
  if (pl->n_cand == 0 || !pl->n_inst || !pl->tp_idx || !pl->max_batch || !pl->occ || !pl->q_ticks)
    return MAASO_E_INVALID_ARG;
  if (pl->i_pad == 0 || pl->i_pad > MAASO_MAX_INSTANCES) return MAASO_E_SHAPE;
  if (rq->n_req != 0 && (!rq->prompt_len || !rq->out_len || !rq->slo_class))
    return MAASO_E_INVALID_ARG;
  if (rq->n_req > MAASO_MAX_REQUESTS) return MAASO_E_SHAPE;
  if (!(prm->s_bar > 0.0f) || !std::isfinite(prm->s_bar)) return MAASO_E_INVALID_ARG;
  if (!(prm->pen_kappa >= 0.0f) || !std::isfinite(prm->pen_kappa)) return MAASO_E_INVALID_ARG;
  if (prm->tbt_mode > 1u || prm->policy > 1u) return MAASO_E_INVALID_ARG;
  return MAASO_OK;
}

ModelParams model_params(const maaso_ctx* ctx, const maaso_params* prm) {
  ModelParams mp;
  mp.s_bar = prm->s_bar;
  mp.pen_kappa = prm->pen_kappa;
  mp.tbt_mode = prm->tbt_mode;
  mp.n_tp = ctx->n_tp;
  mp.b_cap = ctx->b_cap;
  return mp;
}

// AdmissionBounds::narrow (per_window = 0) and narrow_queue.  The occupancy penalty is at most 1 + pen_kappa;
// a finite service time leaves no 0 * inf in a wait.  An instance admits while its wait is within the
// largest first-token deadline D, and so is each prefill: its queue ends a window below D * (1 + window).
// narrow_queue also takes a service time that is not zero in binary32: NarrowSequence lets no time pass behind the
// last window and relies on nothing completing in none.
bool narrow_ticks(const maaso_ctx* ctx, const maaso_params* prm, uint64_t per_window) {
  double d = 0.0;
  for (uint32_t k = 0; k < ctx->n_slo; ++k) d = std::max(d, (double)ctx->d_ttft[k]);
  return d < (double)kNarrowSeconds && d * (1.0 + (double)per_window) < 4095.0 &&
         (double)prm->s_bar * (double)ctx->tbt_max * (1.0 + (double)prm->pen_kappa) < 1e38;
}

AdmissionBounds admission_bounds(const maaso_ctx* ctx, const maaso_params* prm) {
  AdmissionBounds b{0.0f, 0.0f, 0.0f, 0.0f, false, false};
  for (uint32_t k = 0; k < ctx->n_slo; ++k) {
    b.d_ttft = std::max(b.d_ttft, ctx->d_ttft[k]);
    b.d_tbt = std::max(b.d_tbt, ctx->d_tbt[k]);
  }
  b.e_ttft = b.d_ttft * 0x1p-20f;
  b.e_tbt = b.d_tbt * 0x1p-20f;
  b.narrow = narrow_ticks(ctx, prm, 0u);
  b.narrow_queue = (double)prm->s_bar * (double)ctx->tbt_min >= (double)FLT_MIN &&
                   narrow_ticks(ctx, prm, prm->window ? prm->window : MAASO_MAX_REQUESTS);
  return b;
}

int score_assign_impl(maaso_ctx* ctx, const maaso_placements* pl, const uint32_t* cand_sel,
                      const maaso_requests* rq, const maaso_params* prm, const maaso_assign_out* out,
                      void* hip_stream);

int placement_sweep_impl(maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                         const maaso_params* prm, uint32_t* sat_count, float* sat_ratio,
                         uint32_t* best_cand, void* hip_stream, bool static_scratch);

void fill_assign_args(AssignArgs& a, const maaso_ctx* ctx, const maaso_placements* pl,
                      const maaso_requests* rq, const maaso_params* prm,
                      const maaso_assign_out* out) {
  a.tab = ctx->tab;
  a.cells = ctx->cells;
  a.mp = model_params(ctx, prm);
  a.n_slo = ctx->n_slo;
  std::memcpy(a.d_ttft, ctx->d_ttft, sizeof(a.d_ttft));
  std::memcpy(a.d_tbt, ctx->d_tbt, sizeof(a.d_tbt));
  std::memcpy(a.i_ttft, ctx->i_ttft, sizeof(a.i_ttft));
  std::memcpy(a.i_tbt, ctx->i_tbt, sizeof(a.i_tbt));
  a.i_pad = pl->i_pad;
  a.n_cand = pl->n_cand;
  a.cand_sel = nullptr;
  a.n_inst = pl->n_inst;
  a.tp_idx = pl->tp_idx;
  a.max_batch = pl->max_batch;
  a.occ = pl->occ;
  a.q_ticks = reinterpret_cast<uint64_t*>(pl->q_ticks);
  a.n_req = rq->n_req;
  a.prompt_len = rq->prompt_len;
  a.out_len = rq->out_len;
  a.slo_class = rq->slo_class;
  a.arrival_ticks = rq->arrival_ticks;
  a.chosen = out->chosen;
  a.slack = out->slack;
  a.ttft = out->ttft;
  a.tbt = out->tbt;
  a.e2e = out->e2e;
  a.n_satisfied = reinterpret_cast<unsigned long long*>(out->n_satisfied);
  a.status = ctx->status;
  a.bounds = admission_bounds(ctx, prm);
  a.sat_acc = reinterpret_cast<unsigned long long*>(ctx->status + kSatWord);
}

// Wavefronts per candidate and requests per lane of the windowed sweep.  One wavefront per candidate wastes
// least (state, evaluation and the choice of admissible instances are per wavefront) once there are
// enough candidates to fill the device, and where a window is no more than its lanes; four shorten the walk
// through the windows where they are not.
// Measured, four wavefronts' time over one's, 4 / 32 / 256 slots: 400 candidates, windows of 80: 1.16 / 0.98 / 0.90; 780, of
// 256: 1.43 / 1.08 / 0.92, of 512: 1.40 / 0.93 / 0.85; 1024, of 512: 1.41 / 0.94 / 0.92, of 1000: 1.34 / 0.83 / 0.81, of 2000:
// 0.97 / 0.65 / 0.65; 1500, of 1000: 1.53 / 0.88 / 1.03, of 2000: 1.30 / 0.78 / 0.78; 3000, of 2000: 1.82 / 1.07 / 1.02, of 8000:
// 1.16 / 0.84 / 0.94; 8192 of 4096: 1.4.  The line, units * units / 2048, runs between.
// Requests per lane: as many as a window has for one pass (2000 candidates, 128 slots, 1 / 2 / 4: windows of 64
// 0.73 / 0.78 / 0.88 ms, of 128 0.53 / 0.47 / 0.53 ms, of 192 0.44 / 0.42 / 0.37 ms, of 256
// 0.42 / 0.35 / 0.30 ms); with four wavefronts one up to windows of 1024.
template <bool kScore, bool kSQ, int S>
void launch_sweep_window_s(const SweepWindowArgs& a, uint64_t per_window, size_t lds, hipStream_t s) {
  const uint64_t units = (uint64_t)a.n_cand * a.n_sets;
  const bool alone = units >= 4096u || per_window <= 64u || per_window <= units * units / 2048u;
  const dim3 b(kAssignThreads);
  const dim3 g((alone ? (a.n_cand + 3u) / 4u : a.n_cand) * a.n_sets);
  if (alone) {
    if (per_window > 128u) hipLaunchKernelGGL((sweep_window_kernel<kScore, S, 1, 4, kSQ>), g, b, lds, s, a);
    else if (per_window > 64u) hipLaunchKernelGGL((sweep_window_kernel<kScore, S, 1, 2, kSQ>), g, b, lds, s, a);
    else hipLaunchKernelGGL((sweep_window_kernel<kScore, S, 1, 1, kSQ>), g, b, lds, s, a);
  } else {
    if (per_window >= 1024u) hipLaunchKernelGGL((sweep_window_kernel<kScore, S, 4, 4, kSQ>), g, b, lds, s, a);
    else hipLaunchKernelGGL((sweep_window_kernel<kScore, S, 4, 1, kSQ>), g, b, lds, s, a);
  }
}

// The windows that a block per candidate (sweep_block_kernel) takes where there are few candidates.  Measured, the
// forms chosen otherwise against it, 24 windows, mixed instances / jittered profiles and loaded instances:
//   16 candidates, 16 slots, windows of 3, 5, 64, 256, 320: 0.99/0.97, 1.38/1.37, 1.78/1.80, 1.16/1.15, 0.89/0.91 times its
//   time; 8 slots, 512: 0.96/0.95 (fresh jittered instances: 1.2); 128 slots, 64, 128, 192: 1.75/2.97, 1.24/1.61, 0.78/0.96;
//   768: 32 slots, 5, 64, 256, 320: 1.16/1.20, 1.77/1.99, 1.09/1.20, 0.87/0.91; 256 slots, 128, 192: 1.16/1.60, 0.68/0.86;
//   1024: 16 slots, 64, 128, 192: 1.37/1.51, 1.09/1.15, 0.93/0.92; 128 slots, 64, 96: 1.20/2.06, 0.86/1.28;
//   1536: 64 slots, 5, 12, 64, 96: 0.86/0.86, 1.70/1.75, 1.23/1.66, 0.91/1.30; 2048: 12, 32, 48: 1.27/1.33, 1.24/1.76, 0.94/1.37,
//   8 slots, 12: 0.94/0.97.
// Shortest queue (loaded / jittered): 768 candidates, 8 slots, 64, 128, 256: 0.91/0.91, 1.08/1.10, 0.98/1.02; 32 slots, 128,
// 192: 1.14/1.29, 0.89/1.03; 128 slots, 64, 96: 0.90/1.29, 0.85/1.21; 1024: 8 slots, 24, 48: 1.11/1.09, 0.96/0.94; 1536: 0.74/0.75.
struct BlockWindows {
  uint64_t shortest, longest;
};
BlockWindows block_windows(uint64_t blocks, uint32_t i_pad, bool shortest_queue) {
  if (shortest_queue) {
    if (blocks <= 768u) return {1u, i_pad <= 8u ? 256u : i_pad <= 32u ? 128u : 64u};
    return {1u, blocks <= 1280u ? 32u : 0u};
  }
  if (blocks <= 768u) return {5u, i_pad <= 8u ? 512u : i_pad <= 64u ? 256u : 128u};
  if (blocks <= 1024u) return {5u, i_pad > 12u && i_pad <= 64u ? 128u : 64u};
  if (blocks <= 1536u) return {7u, 64u};
  return {9u, blocks <= 2560u && i_pad > 12u ? 32u : 0u};
}

inline size_t up256(size_t x) { return (x + 255) & ~size_t(255); }

// Where a launch over windows keeps its requests laid out by class and length (ordered_windows.hpp), in a workspace.
struct OrderedPlan {
  OrderArgs order;
  OrderedSets sets;
  uint32_t blocks;   // of the launch that lays them out
  uint32_t threads;
  size_t lds, bytes;
};

// Of request set `t`, of which n_windows windows are laid out at `at` (moved behind them).
OrderedSet plan_set(const SweepWindowSet& t, uint32_t n_slo, uint32_t size_log2, uint64_t n_windows, unsigned char*& at) {
  const uint32_t per_window = std::min(t.window, t.n_req);
  OrderedSet o;
  o.segments = (per_window + kSegment - 1u) / kSegment;
  o.size_log2 = size_log2;
  o.batches = o.segments * segment_batches(std::min(per_window, kSegment), n_slo, 1u << size_log2);
  auto take = [&](size_t bytes) {
    unsigned char* p = at;
    at += up256(bytes);
    return p;
  };
  const size_t slots = (size_t)n_windows * o.batches << size_log2;
  o.len = reinterpret_cast<float*>(take(slots * sizeof(float)));
  o.out = reinterpret_cast<float*>(take(slots * sizeof(float)));
  o.batch = reinterpret_cast<Batch*>(take((size_t)n_windows * o.batches * sizeof(Batch)));
  o.gap = reinterpret_cast<uint32_t*>(take((size_t)n_windows * sizeof(uint32_t)));
  return o;
}

// All sets of `a` from `from` on (null: how much that is, alone); false where there is no room for them.
bool plan_ordered(const SweepWindowArgs& a, uint32_t size_log2, unsigned char* from, size_t room, OrderedPlan& plan) {
  plan.sets.ticks = nullptr;
  plan.sets.row_ticks = 0u;
  plan.order.n_slo = a.n_slo;
  plan.order.status = a.status;
  plan.order.n_sets = a.n_sets;
  unsigned char* at = from;
  uint64_t blocks = 0;
  uint32_t segment = 1u;
  for (uint32_t k = 0; k < a.n_sets; ++k) {
    const SweepWindowSet& t = a.sets[k];
    const uint64_t n_windows = ((uint64_t)t.n_req + t.window - 1u) / t.window;
    plan.order.first[k] = (uint32_t)blocks;
    plan.order.sets[k] = t;
    plan.order.to[k] = plan.sets.set[k] = plan_set(t, a.n_slo, size_log2, n_windows, at);
    blocks += n_windows * plan.order.to[k].segments;
    if (blocks > 1u << 24) return false;
    segment = std::max(segment, std::min(std::min(t.window, t.n_req), kSegment));
  }
  plan.blocks = (uint32_t)blocks;
  plan.threads = segment <= 256u * kOrderPer ? 256u : 1024u;
  plan.lds = order_lds(segment, a.n_slo, 1u << size_log2);
  plan.bytes = (size_t)(at - from);
  return up256(plan.bytes) <= room && plan.bytes < (size_t)1 << 32;
}

// The windowed sweep of every (request set, candidate); shapes are chosen by the set with the longest
// windows (the choice never changes a result).
template <bool kScore, bool kSQ>
int launch_sweep_window_v(const SweepWindowArgs& a, size_t lds, uint32_t n_cu, unsigned char* end, size_t room, hipStream_t s) {
  uint64_t per_window = 0, n_windows = 0;
  for (uint32_t k = 0; k < a.n_sets; ++k) {
    const uint64_t pw = a.sets[k].window < a.sets[k].n_req ? a.sets[k].window : a.sets[k].n_req;
    if (pw > per_window) per_window = pw;
    n_windows = std::max(n_windows, ((uint64_t)a.sets[k].n_req + a.sets[k].window - 1u) / a.sets[k].window);
  }
  const uint64_t blocks = (uint64_t)a.n_cand * a.n_sets;
  if (blocks == 0 || blocks > 0x7fffffffull) return MAASO_E_SHAPE;
  // Laid out by class and length: in batches of 16 where a window then is two groups at most, else of 64 (8192 candidates,
  // windows of 4096, batches of 32: 2 % slower).  The kernels below where there is no room, and in a captured launch, which may
  // replay while another call has its requests laid out.
  OrderedPlan plan;
  const bool small = per_window <= kSegment && segment_batches((uint32_t)per_window, a.n_slo, 16u) <= 32u;
  if (end && a.bounds.narrow && sweep_lays_out(blocks, a.n_sets, a.i_pad, per_window, n_windows, kSQ) &&
      plan_ordered(a, small ? 4u : 6u, nullptr, room, plan) && !is_captured(s)) {
    TicksArgs t;
    t.n_batches = (uint32_t)(((uint64_t)a.sets[0].n_req + a.sets[0].window - 1u) / a.sets[0].window) * plan.sets.set[0].batches;
    const uint64_t with_table = up256(plan.bytes) + (uint64_t)t.n_batches * a.cells * sizeof(uint32_t);
    const bool table = !small && a.n_sets == 1u && sweep_sums_batches(a.i_pad, per_window, n_windows) && up256(with_table) <= room;
    unsigned char* at = end - up256(table ? (size_t)with_table : plan.bytes);
    plan_ordered(a, small ? 4u : 6u, at, room, plan);
    hipLaunchKernelGGL(order_requests_kernel, dim3(plan.blocks), dim3(plan.threads), plan.lds, s, plan.order);
    const dim3 g((a.n_cand + 3u) / 4u * a.n_sets), b(kAssignThreads);
    if (table) {
      t.tab = a.tab;
      t.cells = a.cells;
      t.len = plan.sets.set[0].len;
      t.batch = plan.sets.set[0].batch;
      t.ticks = reinterpret_cast<uint32_t*>(at + up256(plan.bytes));
      plan.sets.ticks = t.ticks;
      plan.sets.row_ticks = t.n_batches;
      hipLaunchKernelGGL(batch_ticks_kernel, dim3((t.n_batches / 4u + 3u) / 4u, (a.cells + 63u) / 64u), dim3(256), 0, s, t);
    }
    auto launch = [&](auto s_) {
      if (small) hipLaunchKernelGGL((sweep_ordered_kernel<kScore, s_(), 4, true, kSQ, false>), g, b, lds, s, a, plan.sets);
      else if (table) hipLaunchKernelGGL((sweep_ordered_kernel<kScore, s_(), 6, false, kSQ, true>), g, b, lds, s, a, plan.sets);
      else hipLaunchKernelGGL((sweep_ordered_kernel<kScore, s_(), 6, false, kSQ, false>), g, b, lds, s, a, plan.sets);
    };
    if (a.i_pad <= 64u) launch(std::integral_constant<int, 1>{});
    else if (a.i_pad <= 128u) launch(std::integral_constant<int, 2>{});
    else launch(std::integral_constant<int, 4>{});
    return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
  }
  const BlockWindows bw = block_windows(blocks, a.i_pad, kSQ);
  if (per_window >= bw.shortest && per_window <= bw.longest) {
    uint32_t lpr_log2 = 0;  // lanes per request: as many as a pass over the window has, while a lane walks more than one trip
    while (lpr_log2 < kMaxLprLog2 && (per_window << (lpr_log2 + 1u)) <= (uint64_t)kBlockThreads && (kBlockTrip << lpr_log2) < a.i_pad)
      ++lpr_log2;
    hipLaunchKernelGGL((sweep_block_kernel<kScore, kSQ>), dim3((uint32_t)blocks), dim3(kBlockThreads), lds, s, a, lpr_log2);
    return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
  }
  // Short windows go to the kernel whose lanes are the instances (the block form ahead of it takes few candidates).
  const uint32_t short_window = sweep_short_window(a.i_pad, kScore, a.bounds.narrow_queue);
  bool one_by_one = !kSQ;
  for (uint32_t k = 0; k < a.n_sets; ++k) one_by_one = one_by_one && a.sets[k].window <= short_window;
  if (one_by_one) {
    const size_t lds_seq = ((size_t)a.cells + 1u) * sizeof(float4);  // one more row: slots without an instance
    // Wavefronts per block: eight (tables and requests shared by more, 2 to 3 % faster where both spread as well), four
    // where that leaves fewer on the fullest compute unit and the tables leave room for its blocks.  64 slots, eight / four, us:
    // 3000 candidates one by one 73.5 / 66.2, windows of 3: 69.4 / 64.3; 5000: 92.6 / 84.8; 9000: 140 / 132; 128 slots, 6000: 128 / 132;
    // 8192: 158 / 161, with tables of 1028 cells (seven blocks of four at a time) 159 / 173.
    auto fullest = [&](uint32_t waves) {  // blocks on it
      return ((uint64_t)((a.n_cand + waves - 1u) / waves) * a.n_sets + n_cu - 1u) / n_cu;
    };
    const uint32_t fit = std::min(kSeqLds / (uint32_t)(lds_seq + kSeqShared), 8u);
    const bool four = a.i_pad > 128u || (fullest(4u) < 2u * fullest(8u) && (fit == 8u || fullest(4u) <= fit));
    const uint32_t per_block = four ? 4u : kSeqThreads / 64;
    const dim3 g((a.n_cand + per_block - 1u) / per_block * a.n_sets);
    bool one = true;  // every set request by request
    for (uint32_t k = 0; k < a.n_sets; ++k) one = one && a.sets[k].window == 1u;
    if constexpr (!kSQ) {
      const dim3 b(per_block * 64u);
      auto launch = [&](auto s_, auto one_, auto fits_) {
        hipLaunchKernelGGL((sweep_seq_kernel<kScore, s_(), one_(), fits_()>), g, b, lds_seq, s, a);
      };
      auto by_form = [&](auto s_, auto one_) {
        if (a.bounds.narrow_queue) launch(s_, one_, std::true_type{});
        else launch(s_, one_, std::false_type{});
      };
      auto by_slots = [&](auto one_) {
        if (a.i_pad <= 64u) by_form(std::integral_constant<int, 1>{}, one_);
        else if (a.i_pad <= 128u) by_form(std::integral_constant<int, 2>{}, one_);
        else by_form(std::integral_constant<int, 4>{}, one_);
      };
      if (one) by_slots(std::true_type{});
      else by_slots(std::false_type{});
    }
    return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
  }
  if (a.i_pad <= 64u) launch_sweep_window_s<kScore, kSQ, 1>(a, per_window, lds, s);
  else if (a.i_pad <= 128u) launch_sweep_window_s<kScore, kSQ, 2>(a, per_window, lds, s);
  else launch_sweep_window_s<kScore, kSQ, 4>(a, per_window, lds, s);
  return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
}

template <bool kScore>
int launch_sweep_window(const SweepWindowArgs& a, uint32_t policy, const maaso_ctx* ctx, bool may_lay_out, hipStream_t s) {
  const size_t lds = (size_t)3 * ctx->cells * sizeof(float);  // profile tables
  const uint32_t n_cu = (uint32_t)ctx->n_cu;
  unsigned char* end = may_lay_out ? static_cast<unsigned char*>(ctx->ws) + ctx->ws_bytes : nullptr;  // (whole MiB)
  // (the windowed distributor's profile is read from its start later)
  const size_t low = std::max(ctx->ws_low, ctx->window_profiled ? sizeof(WindowWs) : 0u);
  const size_t room = ctx->ws_bytes - std::min(up256(low), ctx->ws_bytes);
  return policy ? launch_sweep_window_v<kScore, true>(a, lds, n_cu, end, room, s)
                : launch_sweep_window_v<kScore, false>(a, lds, n_cu, end, room, s);
}

// Everything but the request sets.
void fill_sweep_window_args(SweepWindowArgs& a, const maaso_ctx* ctx, const maaso_placements* pl,
                            const maaso_params* prm) {
  a.tab = ctx->tab;
  a.cells = ctx->cells;
  a.mp = model_params(ctx, prm);
  a.n_slo = ctx->n_slo;
  std::memcpy(a.d_ttft, ctx->d_ttft, sizeof(a.d_ttft));
  std::memcpy(a.d_tbt, ctx->d_tbt, sizeof(a.d_tbt));
  std::memcpy(a.i_ttft, ctx->i_ttft, sizeof(a.i_ttft));
  std::memcpy(a.i_tbt, ctx->i_tbt, sizeof(a.i_tbt));
  a.n_cand = pl->n_cand;
  a.i_pad = pl->i_pad;
  a.n_inst = pl->n_inst;
  a.tp_idx = pl->tp_idx;
  a.max_batch = pl->max_batch;
  a.occ = pl->occ;
  a.q_ticks = reinterpret_cast<const uint64_t*>(pl->q_ticks);
  a.bounds = admission_bounds(ctx, prm);
  a.n_sets = 0;
  std::memset(a.sets, 0, sizeof(a.sets));
  a.status = ctx->status;
  a.alpha = a.beta = 0.0f;
  a.gamma_t = a.gamma_l = 1.0f;
}

// Appends a request set.  prm->window == 0 (static) = one window over everything: the state update is
// never reached.
void add_sweep_window_set(SweepWindowArgs& a, const maaso_requests* rq, const maaso_params* prm,
                          uint32_t* sat_count, const maaso_score_out* out) {
  SweepWindowSet& t = a.sets[a.n_sets++];
  t.n_req = rq->n_req;
  t.window = prm->window ? prm->window : (rq->n_req ? rq->n_req : 1u);
  t.prompt_len = rq->prompt_len;
  t.out_len = rq->out_len;
  t.slo_class = rq->slo_class;
  t.arrival_ticks = rq->arrival_ticks;
  t.sat_count = sat_count;
  t.phi_s = out ? out->phi_s : nullptr;
  t.phi_t = out ? out->phi_t : nullptr;
  t.phi_l = out ? out->phi_l : nullptr;
  t.score = out ? out->score : nullptr;
}

// Workspace the static sweep of a shape is charged with: 4 bytes per (class, request), 16 per instance
// slot, and per (request tile, XCD) queue 4 bytes and 16 per block that would serve it, by the launch-shape
// knobs or the rules here.  The sweep has no such tiles, queues or records: it keeps 4 bytes per request.
// The charge is part of the interface - which calls are refused, and what maaso_ctx_reserve reserves - and
// stays what it was, so that a caller's reservations and refusals do not depend on how the sweep works.
int static_sweep_bytes(const maaso_ctx* ctx, uint32_t C, uint32_t I, uint32_t R, size_t& bytes) {
  const uint32_t K = ctx->n_slo;
  uint32_t Q = ctx->sweep_q;
  if (Q == 0) Q = R >= (1u << 17) ? 16u : (R >= (1u << 14) ? 8u : (R >= (1u << 12) ? 4u : 2u));
  uint32_t G = 512u / I;
  if (G > 64u) G = 64u;
  const uint32_t g_want = ctx->sweep_group ? ctx->sweep_group : (256u / I ? 256u / I : 1u);
  if (g_want < G) G = g_want;
  const uint32_t n_items = (C + G - 1) / G;
  const uint32_t tile = (uint32_t)kSweepThreads * Q;
  const uint32_t tiles = (uint32_t)(((uint64_t)R + tile - 1) / tile) + K;
  const uint32_t per_queue = (n_items + 7u) / 8u;
  uint32_t bq = ctx->sweep_blocks_per_queue;
  if (bq == 0) {
    bq = ((uint32_t)ctx->n_cu * 18u + 4u * tiles) / (8u * tiles);
    if (bq == 0) bq = 1;
  }
  if (bq > per_queue) bq = per_queue ? per_queue : 1u;
  const uint64_t blocks64 = (uint64_t)8 * tiles * bq;
  if (blocks64 > 0x7fffffffull) return MAASO_E_SHAPE;
  // (the shapes whose preparation would have taken a grid beyond 2^31 blocks)
  if (((uint64_t)R + 1023u) / 1024u + ((uint64_t)C * I + 511u) / 512u > 0x7fffffffull) return MAASO_E_SHAPE;
  const size_t queue_words = (size_t)tiles * 8u + 4u * (size_t)blocks64;
  bytes = up256((size_t)K * (R ? R : 1u) * sizeof(float)) + up256((size_t)C * I * sizeof(float4)) +
          up256(queue_words * sizeof(uint32_t));
  return MAASO_OK;
}

// Workspace that no call with at most C candidates of I slots and R requests exceeds, whatever launch
// shape it takes with the context's current knobs: the static sweep (its queue part bounded at two
// requests per lane, where the grid has the most request tiles), the windowed distributor's
// accumulators, the split's per-block counts.
size_t workspace_bound(const maaso_ctx* ctx, uint32_t C, uint32_t I, uint32_t R) {
  const uint64_t K = ctx->n_slo;
  const size_t lbuf = up256((size_t)K * (R ? R : 1u) * sizeof(float));
  const size_t recs = up256((size_t)C * I * sizeof(float4));
  const uint64_t nrb = ((uint64_t)R + 2u * kSweepThreads - 1) / (2u * kSweepThreads) + K;
  // blocks = 8 * nrb * bq with bq = floor((18 n_cu + 4 nrb) / (8 nrb)), at least 1
  const uint64_t blocks = ctx->sweep_blocks_per_queue ? 8u * nrb * ctx->sweep_blocks_per_queue
                                                      : (uint64_t)ctx->n_cu * 18u + 12u * nrb;
  const size_t queue = up256((size_t)(nrb * 8u + 4u * blocks) * sizeof(uint32_t));
  size_t need = lbuf + recs + queue;
  if (need < sizeof(WindowWs)) need = sizeof(WindowWs);
  const size_t split = (size_t)(((uint64_t)R + kSplitPerBlock - 1) / kSplitPerBlock + 1u) * sizeof(uint32_t);
  return need < split ? split : need;
}

// The launches of the static sweep; `ws` holds the grouped prompt lengths, 4 bytes per request.
int launch_static_sweep(maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                        const maaso_params* prm, void* ws, size_t ws_bytes, uint32_t* sat_count, float* sat_ratio,
                        uint32_t* best_cand, hipStream_t s) {
  const uint32_t C = pl->n_cand, I = pl->i_pad, K = ctx->n_slo, R = rq->n_req;
  uint32_t* hist = ctx->status + kCounterWord;
  uint32_t* offsets = hist + 2u * kHistWords;
  if (ctx->counters_dirty) {  // an earlier call failed between its launches
    hipLaunchKernelGGL(fill_u32_kernel, dim3(16), dim3(256), 0, s, ctx->status + kTotalsWord,
                       (kCounterWord - kTotalsWord) + 2u * kHistWords, 0u);
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(64), 0, s, ctx->status + kClassWord, (uint32_t)kMaxSlo, 0u);
    if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
    ctx->counters_dirty = false;
  }
  ctx->counters_dirty = true;
  const bool small = R <= kSmallRequests;
  // Few candidates: every block works out all thresholds and compares its share of the requests with them.
  // Grouping first costs two more launches and two passes over the requests instead.  Both in nanoseconds, as
  // fitted to 40 shapes: the one launch by trips of 256 slots (an evaluation per class each), candidates x
  // classes and comparisons; the three by classes and requests.  Measured, one launch against three: 2 candidates
  // x 91 slots x 92,049 requests, sixteen classes: 17.9 / 27.0 us; 16 x 32 x 2,000,000, three: 26.8 / 69; 55 x 17 x 158,856,
  // one: 18.8 / 22.7; 17 x 34 x 310,617, sixteen: 31.0 / 35.0; 91 x 5 x 62,421, sixteen: 30.9 / 22.7; 79 x 41 x 6753, one:
  // 24.7 / 16.9; 63 x 22 x 116,985, three: 23.8 / 21.5; 128 x 4 x 262,144, three: equal.
  const uint64_t few_ns = 9000u + ((uint64_t)C * I + 255u) / 256u * (1100u + 360u * K) + 9u * (uint64_t)C * K / 2u +
                          (uint64_t)C * R / 2500u;
  const uint64_t grouped_ns = 17000u + 200u * K + (uint64_t)R * (260u + 12u * K) / 10000u;
  const bool few = !small && C <= kFewCandidates && few_ns <= grouped_ns;
  // Bins per class: a pass over all groups is most of what the grouping launches cost on some ten thousand
  // requests, so no more than some 256 groups while bins stay below a few hundred requests and the look-ups
  // of all candidates some megabytes (213 candidates x 32 slots x 7112 requests, sixteen classes: 26 -> 20 us;
  // 45 x 34 x 7773: 26.4 -> 19.8).
  LengthGroups groups{K, 0u};
  while (groups.count() > 256u && (uint64_t)R << (groups.shift + 1u) <= (uint64_t)K * kLenBins << 7 &&
         (uint64_t)C * R << (groups.shift + 1u) <= 1ull << 28)
    ++groups.shift;
  const uint32_t n_groups = groups.count();
  // a group of about 512 slots, two per thread, but no fewer than some 1024 groups while there are the
  // candidates for it (four blocks per compute unit)
  uint32_t G = (uint32_t)(((uint64_t)C + 1023u) / 1024u);
  if (G > 512u / I) G = 512u / I;
  if (G > kMaxGroup) G = kMaxGroup;
  if (G == 0u) G = 1u;
  const uint32_t cand_groups = (uint32_t)(((uint64_t)C + G - 1u) / G);
  // Thresholds beside the grouping keep a word per (candidate, class) behind the lengths: where the workspace has
  // room for them (next to any that holds the call's charge; with many classes, few slots and few requests it may not).
  const uint32_t cap = (uint32_t)ctx->n_cu * 6u;  // 65,536 x 32 slots, the same inputs repeated: 33.8 us with 6 blocks per compute unit, 35.1 with 5, 36.4 with 8
  const uint32_t rank_cap = (uint32_t)ctx->n_cu * 8u;
  const size_t at_longest = up256((size_t)R * sizeof(float)), at_pairs = at_longest + up256((size_t)C * K * sizeof(uint32_t));
  const size_t at_best = at_pairs + up256((size_t)rank_cap * 2u * sizeof(uint64_t));
  // (The one-launch form of up to 4096 requests keeps the atomics: settled apart it is 2 to 5 % slower at any size.)
  // A fourth launch to settle the totals costs less than their delivery by atomics from a few hundred blocks on, the
  // thresholds beside the dealing out pay with some 10^5 requests: 64 candidates x 99 slots x 4981 requests: 16.9 us in
  // three launches, 18.2 in four; 67 x 32 x 4775: 17.5 / 18.0; 1039 x 6 x 8704: 18.7 / 18.5; 53 x 59 x 196,187: 26.7 / 24.7;
  // 8974 x 8 x 151,529: 30.2 / 25.7; 59,250 x 3 x 188,741: 64 / 48.
  const size_t with_best = at_best + (size_t)rank_cap * sizeof(uint64_t);
  const bool beside = !small && !few && (C >= 512u || R >= 1u << 16) && with_best <= ws_bytes;
  if (ws == ctx->ws && !small && !few) use_workspace(ctx, beside ? with_best : at_longest, s);
  TimedRegion timed(ctx, s);  // all launches of the call
  if (beside) {
    GroupArgs g;
    g.prompt_len = rq->prompt_len;
    g.slo_class = rq->slo_class;
    g.n_req = R;
    g.groups = groups;
    g.per_block = R > (1u << 20) ? (uint32_t)(((uint64_t)R + 1023u) / 1024u) : 1024u;
    g.hist = hist;
    g.of_class = ctx->status + kClassWord;
    g.cursor = hist + n_groups;
    g.offsets = offsets;
    g.sorted = static_cast<float*>(ws);
    g.status = ctx->status;
    const uint32_t blocks = (uint32_t)(((uint64_t)R + g.per_block - 1) / g.per_block);
    ThresholdArgs t;
    t.tab = ctx->tab;
    t.cells = ctx->cells;
    t.mp = model_params(ctx, prm);
    t.n_slo = K;
    std::memcpy(t.d_ttft, ctx->d_ttft, sizeof(t.d_ttft));
    std::memcpy(t.d_tbt, ctx->d_tbt, sizeof(t.d_tbt));
    t.n_cand = C;
    t.i_pad = I;
    t.n_inst = pl->n_inst;
    t.tp_idx = pl->tp_idx;
    t.max_batch = pl->max_batch;
    t.occ = pl->occ;
    t.q_ticks = reinterpret_cast<const uint64_t*>(pl->q_ticks);
    t.group = G;
    t.longest = reinterpret_cast<uint32_t*>(static_cast<unsigned char*>(ws) + at_longest);
    t.status = ctx->status;
    t.pairs = reinterpret_cast<unsigned long long*>(static_cast<unsigned char*>(ws) + at_pairs);
    t.of_class = ctx->status + kClassWord;
    t.n_groups = cand_groups;
    const size_t lds_g = (size_t)group_lds_words(n_groups) * sizeof(uint32_t);
    const size_t lds = std::max(lds_g, (size_t)G * K * sizeof(uint32_t));
    const bool rows = I % 16u == 0u, whole = groups.shift == 0u;
    const uint32_t t_blocks = std::min(cand_groups, cap);
    const dim3 pg(blocks + t_blocks), pb(kSweepThreads);
    if (whole) hipLaunchKernelGGL(sweep_hist_kernel<true>, dim3(blocks), pb, lds_g, s, g);
    else hipLaunchKernelGGL(sweep_hist_kernel<false>, dim3(blocks), pb, lds_g, s, g);
    if (rows && whole) hipLaunchKernelGGL((sweep_prepare_kernel<true, true>), pg, pb, lds, s, g, t, blocks);
    else if (rows) hipLaunchKernelGGL((sweep_prepare_kernel<true, false>), pg, pb, lds, s, g, t, blocks);
    else if (whole) hipLaunchKernelGGL((sweep_prepare_kernel<false, true>), pg, pb, lds, s, g, t, blocks);
    else hipLaunchKernelGGL((sweep_prepare_kernel<false, false>), pg, pb, lds, s, g, t, blocks);
    RankArgs r;
    r.groups = groups;
    r.n_cand = C;
    r.n_req = R;
    r.longest = t.longest;
    r.of_class = ctx->status + kClassWord;
    r.block_best = reinterpret_cast<unsigned long long*>(static_cast<unsigned char*>(ws) + at_best);
    r.offsets = offsets;
    r.sorted = g.sorted;
    r.clear = hist;
    uint32_t RG = (uint32_t)(((uint64_t)C + 2047u) / 2048u);
    if (RG > kMaxGroup) RG = kMaxGroup;
    r.group = RG;
    r.n_groups = (uint32_t)(((uint64_t)C + RG - 1u) / RG);
    r.sat_count = sat_count;
    r.sat_ratio = sat_ratio;
    unsigned long long* eval_total = reinterpret_cast<unsigned long long*>(ctx->status + 32);
    const dim3 rg(std::min(r.n_groups, rank_cap));
    const size_t lds_r = ((size_t)n_groups + 1u) * sizeof(uint32_t);
    if (whole) hipLaunchKernelGGL(sweep_rank_kernel<true>, rg, dim3(kSweepThreads), lds_r, s, r);
    else hipLaunchKernelGGL(sweep_rank_kernel<false>, rg, dim3(kSweepThreads), lds_r, s, r);
    hipLaunchKernelGGL(sweep_settle_kernel, dim3(1), dim3(1024), 0, s, r.block_best, rg.x, t.pairs, t_blocks, best_cand, eval_total);
    ctx->last_evaluated = eval_total;
    if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
    ctx->counters_dirty = false;
    return MAASO_OK;
  }
  const size_t lds_g = (size_t)group_lds_words(n_groups) * sizeof(uint32_t);
  if (!small && !few) {
    GroupArgs g;
    g.prompt_len = rq->prompt_len;
    g.slo_class = rq->slo_class;
    g.n_req = R;
    g.groups = groups;
    // 1024 requests a block fill the chip from 2^18 on; beyond 1024 blocks each takes more
    g.per_block = R > (1u << 20) ? (uint32_t)(((uint64_t)R + 1023u) / 1024u) : 1024u;
    g.hist = hist;
    g.of_class = nullptr;
    g.cursor = hist + n_groups;
    g.offsets = offsets;
    g.sorted = static_cast<float*>(ws);
    g.status = ctx->status;
    const uint32_t blocks = (uint32_t)(((uint64_t)R + g.per_block - 1) / g.per_block);
    if (groups.shift == 0u) {
      hipLaunchKernelGGL(sweep_hist_kernel<true>, dim3(blocks), dim3(kSweepThreads), lds_g, s, g);
      hipLaunchKernelGGL(sweep_scatter_kernel<true>, dim3(blocks), dim3(kSweepThreads), lds_g, s, g);
    } else {
      hipLaunchKernelGGL(sweep_hist_kernel<false>, dim3(blocks), dim3(kSweepThreads), lds_g, s, g);
      hipLaunchKernelGGL(sweep_scatter_kernel<false>, dim3(blocks), dim3(kSweepThreads), lds_g, s, g);
    }
    if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
  }
  CountArgs a;
  a.tab = ctx->tab;
  a.cells = ctx->cells;
  a.mp = model_params(ctx, prm);
  a.groups = groups;
  std::memcpy(a.d_ttft, ctx->d_ttft, sizeof(a.d_ttft));
  std::memcpy(a.d_tbt, ctx->d_tbt, sizeof(a.d_tbt));
  a.n_cand = C;
  a.i_pad = I;
  a.n_inst = pl->n_inst;
  a.tp_idx = pl->tp_idx;
  a.max_batch = pl->max_batch;
  a.occ = pl->occ;
  a.q_ticks = reinterpret_cast<const uint64_t*>(pl->q_ticks);
  a.n_req = R;
  a.prompt_len = rq->prompt_len;
  a.slo_class = rq->slo_class;
  a.offsets = offsets;
  a.sorted = static_cast<const float*>(ws);
  a.clear = hist;
  a.group = G;
  a.n_groups = cand_groups;
  a.sat_count = sat_count;
  a.sat_ratio = sat_ratio;
  a.best_cand = best_cand;
  a.totals = reinterpret_cast<SweepTotals*>(ctx->status + kTotalsWord);
  a.eval_total = reinterpret_cast<unsigned long long*>(ctx->status + 32);
  a.status = ctx->status;
  const dim3 grid(a.n_groups < cap ? a.n_groups : cap), block(kSweepThreads);
  const size_t lds = ((size_t)n_groups + 1u) * sizeof(uint32_t);
  if (few) {
    const uint32_t tiles = (R + 1023u) / 1024u;  // four requests a thread
    hipLaunchKernelGGL(sweep_few_kernel, dim3(std::min(tiles, (uint32_t)ctx->n_cu * 4u)), block, 0, s, a);
  } else if (small) {
    if (I % 16u == 0u) hipLaunchKernelGGL((sweep_count_kernel<true, true, false>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((sweep_count_kernel<true, false, false>), grid, block, lds, s, a);
  } else if (groups.shift == 0u) {
    if (I % 16u == 0u) hipLaunchKernelGGL((sweep_count_kernel<false, true, true>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((sweep_count_kernel<false, false, true>), grid, block, lds, s, a);
  } else {
    if (I % 16u == 0u) hipLaunchKernelGGL((sweep_count_kernel<false, true, false>), grid, block, lds, s, a);
    else hipLaunchKernelGGL((sweep_count_kernel<false, false, false>), grid, block, lds, s, a);
  }
  ctx->last_evaluated = a.eval_total;
  if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
  ctx->counters_dirty = false;
  return MAASO_OK;
}

bool score_weights_ok(const maaso_score_weights* wts) {
  return wts && std::isfinite(wts->alpha) && std::isfinite(wts->beta) && wts->gamma_t > 0.0f &&
         wts->gamma_l > 0.0f && std::isfinite(wts->gamma_t) && std::isfinite(wts->gamma_l);
}

// One request set of a scoring launch: where it comes from, where its results go, and - for a side
// of a split that only the device knows - the word holding the split position and which side.
struct ScoreSet {
  const maaso_requests* rq;
  const maaso_score_out* out;
  const uint32_t* split_at;
  uint32_t side;
};

int check_score_sets(const maaso_ctx* ctx, const maaso_placements* pl, uint32_t n_sets,
                     const ScoreSet* sets, const maaso_params* prm, const maaso_score_weights* wts) {
  for (uint32_t k = 0; k < n_sets; ++k) {
    const int rc = check_common(ctx, pl, sets[k].rq, prm);
    if (rc != MAASO_OK) return rc;
    if (!sets[k].out->sat_count || !sets[k].out->score) return MAASO_E_INVALID_ARG;
    if (prm->window != 0u && sets[k].rq->n_req != 0 && !sets[k].rq->arrival_ticks)
      return MAASO_E_INVALID_ARG;
  }
  return score_weights_ok(wts) ? MAASO_OK : MAASO_E_INVALID_ARG;
}

// Scores every candidate against every set in one launch (arguments checked, call guarded).
int launch_score_sets(maaso_ctx* ctx, const maaso_placements* pl, uint32_t n_sets,
                      const ScoreSet* sets, const maaso_params* prm, const maaso_score_weights* wts,
                      hipStream_t s) {
  SweepWindowArgs a;
  fill_sweep_window_args(a, ctx, pl, prm);
  // longest set first: its blocks run longest, so they should start first (a side of a device-side
  // split counts with the size of the whole, its upper bound)
  uint32_t order[MAASO_MAX_REQUEST_SETS];
  for (uint32_t k = 0; k < n_sets; ++k) order[k] = k;
  std::stable_sort(order, order + n_sets,
                   [&](uint32_t x, uint32_t y) { return sets[x].rq->n_req > sets[y].rq->n_req; });
  for (uint32_t k = 0; k < n_sets; ++k) {
    const ScoreSet& t = sets[order[k]];
    add_sweep_window_set(a, t.rq, prm, t.out->sat_count, t.out);
    a.sets[a.n_sets - 1].split_at = t.split_at;
    a.sets[a.n_sets - 1].side = t.side;
  }
  a.alpha = wts->alpha;
  a.beta = wts->beta;
  a.gamma_t = wts->gamma_t;
  a.gamma_l = wts->gamma_l;
  {
    TimedRegion timed(ctx, s);
    const int rc = launch_sweep_window<true>(a, prm->policy, ctx, true, s);
    if (rc != MAASO_OK) return rc;
  }
  for (uint32_t k = 0; k < n_sets; ++k)
    if (sets[k].out->best_cand) {
      hipLaunchKernelGGL(score_argmax_kernel, dim3(1), dim3(1024), 0, s, sets[k].out->score,
                         pl->n_cand, sets[k].out->best_cand);
      if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
    }
  return MAASO_OK;
}

int check_split(const maaso_ctx* ctx, const maaso_requests* rq, const uint32_t* prompt_len_out,
                const uint32_t* out_len_out, const uint8_t* slo_class_out,
                const uint32_t* arrival_ticks_out, const uint32_t* n_tight) {
  if (!ctx || !rq || !n_tight) return MAASO_E_INVALID_ARG;
  if (rq->n_req > MAASO_MAX_REQUESTS) return MAASO_E_SHAPE;
  if (rq->n_req != 0 && (!rq->prompt_len || !rq->out_len || !rq->slo_class || !prompt_len_out ||
                         !out_len_out || !slo_class_out))
    return MAASO_E_INVALID_ARG;
  if (rq->n_req != 0 && rq->arrival_ticks && !arrival_ticks_out) return MAASO_E_INVALID_ARG;
  const uint32_t n_blocks = (uint32_t)(((uint64_t)rq->n_req + kSplitPerBlock - 1) / kSplitPerBlock);
  return need_workspace(ctx, (size_t)(n_blocks ? n_blocks : 1u) * sizeof(uint32_t));
}

// Per-block counts, their scan, the scatter: three launches (arguments checked, call guarded).
int launch_split(maaso_ctx* ctx, const maaso_requests* rq, uint32_t tight_classes,
                 uint32_t* prompt_len_out, uint32_t* out_len_out, uint8_t* slo_class_out,
                 uint32_t* arrival_ticks_out, uint32_t* n_tight, hipStream_t s) {
  const uint32_t n_blocks = (uint32_t)(((uint64_t)rq->n_req + kSplitPerBlock - 1) / kSplitPerBlock);
  SplitArgs a;
  a.n_req = rq->n_req;
  a.prompt_len = rq->prompt_len;
  a.out_len = rq->out_len;
  a.slo_class = rq->slo_class;
  a.arrival_ticks = rq->arrival_ticks;
  a.tight_classes = tight_classes;
  a.n_slo = ctx->n_slo;
  use_workspace(ctx, ((size_t)n_blocks + 1u) * sizeof(uint32_t), s);
  a.block_tight = static_cast<uint32_t*>(ctx->ws);
  a.n_tight = n_tight;
  a.prompt_out = prompt_len_out;
  a.out_len_out = out_len_out;
  a.class_out = slo_class_out;
  a.arrival_out = arrival_ticks_out;
  a.status = ctx->status;
  if (n_blocks) hipLaunchKernelGGL(split_count_kernel, dim3(n_blocks), dim3(kPartitionThreads), 0, s, a);
  hipLaunchKernelGGL(split_scan_kernel, dim3(1), dim3(kPartitionThreads), 0, s, a.block_tight, n_blocks,
                     n_tight);
  if (n_blocks) hipLaunchKernelGGL(split_scatter_kernel, dim3(n_blocks), dim3(kPartitionThreads), 0, s, a);
  return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
}

int check_select(const maaso_ctx* ctx, const maaso_placements* pl, const float* score, uint32_t n_gpus,
                 const float* phi_star, const int32_t* cand_star) {
  if (!ctx || !pl || !score || !phi_star || !cand_star) return MAASO_E_INVALID_ARG;
  if (pl->n_cand == 0 || !pl->n_inst || !pl->tp_idx) return MAASO_E_INVALID_ARG;
  if (!ctx->has_degree) return MAASO_E_INVALID_ARG;
  if (pl->i_pad == 0 || pl->i_pad > MAASO_MAX_INSTANCES || n_gpus > MAASO_MAX_GPUS) return MAASO_E_SHAPE;
  return MAASO_OK;
}

// Alg. 1's selection over n_lists score lists of the same deployments, one block each.
int launch_select(maaso_ctx* ctx, const maaso_placements* pl, uint32_t n_lists, const float* const* score,
                  const uint32_t* chain_offsets, uint32_t n_chains, uint32_t n_gpus,
                  float* const* phi_star, int32_t* const* cand_star, hipStream_t s) {
  SelectArgs a;
  a.n_lists = n_lists;
  for (uint32_t l = 0; l < (uint32_t)kMaxSelectLists; ++l) {
    a.score[l] = l < n_lists ? score[l] : nullptr;
    a.phi_star[l] = l < n_lists ? phi_star[l] : nullptr;
    a.cand_star[l] = l < n_lists ? cand_star[l] : nullptr;
  }
  a.n_cand = pl->n_cand;
  a.i_pad = pl->i_pad;
  a.n_inst = pl->n_inst;
  a.tp_idx = pl->tp_idx;
  a.tp_degree = reinterpret_cast<const uint32_t*>(ctx->tab + (size_t)3 * ctx->cells);
  a.n_tp = ctx->n_tp;
  a.chain_offsets = chain_offsets;
  a.n_chains = chain_offsets ? n_chains : 0u;
  a.n_gpus = n_gpus;
  a.status = ctx->status;
  hipLaunchKernelGGL(ins_deploy_select_kernel, dim3(n_lists), dim3(kPartitionThreads),
                     ((size_t)n_gpus + 1) * sizeof(unsigned long long), s, a);
  return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
}

}  // namespace

extern "C" {

const char* maaso_strerror(int status) {
  switch (status) {
    case MAASO_OK: return "ok";
    case MAASO_E_INVALID_ARG: return "invalid argument";
    case MAASO_E_SHAPE: return "size beyond the library's limits";
    case MAASO_E_TABLE: return "profile table or deadline entry not finite and positive";
    case MAASO_E_HIP: return "HIP runtime error";
    case MAASO_E_NOMEM: return "out of memory";
    case MAASO_E_TIMEOUT: return "inter-window wait timed out on the device";
    case MAASO_E_WORKSPACE: return "workspace too small for this shape: call maaso_ctx_reserve first";
    case MAASO_E_BUSY: return "the context is in use by another call";
    case MAASO_E_RESIDENCY: return "the windowed distributor's blocks cannot all be resident on the device";
    default: return "unknown status";
  }
}

int maaso_profile_tables_load(const maaso_profile_desc* d, int device, maaso_ctx** out_ctx) {
  if (out_ctx) *out_ctx = nullptr;
  if (!d || !out_ctx || !d->prefill_a || !d->prefill_p || !d->tbt || !d->d_ttft || !d->d_tbt)
    return MAASO_E_INVALID_ARG;
  if (d->n_tp == 0 || d->b_cap == 0 || d->n_slo == 0) return MAASO_E_INVALID_ARG;
  if (d->n_slo > MAASO_MAX_SLO || d->b_cap > 65535u) return MAASO_E_SHAPE;
  const uint64_t cells64 = (uint64_t)d->n_tp * ((uint64_t)d->b_cap + 1u);
  if (cells64 > MAASO_MAX_TABLE_CELLS) return MAASO_E_SHAPE;
  const uint32_t cells = (uint32_t)cells64;
  for (uint32_t t = 0; t < d->n_tp; ++t)
    for (uint32_t b = 1; b <= d->b_cap; ++b) {
      const size_t i = (size_t)t * (d->b_cap + 1u) + b;
      const float v[3] = {d->prefill_a[i], d->prefill_p[i], d->tbt[i]};
      for (float x : v)
        if (!(x > 0.0f) || !std::isfinite(x)) return MAASO_E_TABLE;
    }
  for (uint32_t k = 0; k < d->n_slo; ++k) {
    const float v[2] = {d->d_ttft[k], d->d_tbt[k]};
    for (float x : v)
      if (!(x >= 0x1p-20f) || !(x <= 0x1p20f)) return MAASO_E_TABLE;
  }

  int n_dev = 0;
  if (!hip_ok(hipGetDeviceCount(&n_dev)) || device < 0 || device >= n_dev) return MAASO_E_HIP;
  DeviceGuard guard(device);
  if (!guard.ok) return MAASO_E_HIP;

  maaso_ctx* ctx = new (std::nothrow) maaso_ctx();  // value-initialised: every member starts at zero
  if (!ctx) return MAASO_E_NOMEM;
  ctx->device = device;
  ctx->n_tp = d->n_tp;
  ctx->b_cap = d->b_cap;
  ctx->cells = cells;
  ctx->n_slo = d->n_slo;
  ctx->spin_limit = 1u << 22;
  ctx->tbt_min = INFINITY;
  for (uint32_t t = 0; t < d->n_tp; ++t)
    for (uint32_t b = 1; b <= d->b_cap; ++b) {
      const float tbt = d->tbt[(size_t)t * (d->b_cap + 1u) + b];
      ctx->tbt_min = std::min(ctx->tbt_min, tbt);
      ctx->tbt_max = std::max(ctx->tbt_max, tbt);
    }
  for (uint32_t k = 0; k < kMaxSlo; ++k) {
    const bool live = k < d->n_slo;
    ctx->d_ttft[k] = live ? d->d_ttft[k] : 1.0f;
    ctx->d_tbt[k] = live ? d->d_tbt[k] : 1.0f;
    // reciprocal of a deadline: evaluated in double, rounded once to binary32
    ctx->i_ttft[k] = (float)(1.0 / (double)ctx->d_ttft[k]);
    ctx->i_tbt[k] = (float)(1.0 / (double)ctx->d_tbt[k]);
  }
  hipDeviceProp_t prop;
  if (!hip_ok(hipGetDeviceProperties(&prop, device))) { delete ctx; return MAASO_E_HIP; }
  // address of this device's copy of the static scratch array (resolved once per device, with that
  // device current)
  if (device < kMaxDevices) {
    void* sp = g_scratch_ptr[device].load(std::memory_order_acquire);
    if (!sp) {
      if (!hip_ok(hipGetSymbolAddress(&sp, HIP_SYMBOL(scratch))) || !sp) { delete ctx; return MAASO_E_HIP; }
      g_scratch_ptr[device].store(sp, std::memory_order_release);
    }
    ctx->scratch_ptr = sp;
  }
  ctx->n_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;
  ctx->lds_per_block = prop.sharedMemPerBlock;
  if (!hip_ok(hipDeviceGetAttribute(&ctx->cooperative, hipDeviceAttributeCooperativeLaunch, device)))
    ctx->cooperative = 0;
  float* host = static_cast<float*>(std::malloc((size_t)3 * cells * sizeof(float)));
  if (!host) { delete ctx; return MAASO_E_NOMEM; }
  std::memcpy(host, d->prefill_a, (size_t)cells * 4);
  std::memcpy(host + cells, d->prefill_p, (size_t)cells * 4);
  std::memcpy(host + 2 * (size_t)cells, d->tbt, (size_t)cells * 4);
  int rc = MAASO_OK;
  if (!hip_ok(hipMalloc(reinterpret_cast<void**>(&ctx->tab), ((size_t)3 * cells + d->n_tp) * 4)))
    rc = MAASO_E_NOMEM;
  if (rc == MAASO_OK && !hip_ok(hipMalloc(reinterpret_cast<void**>(&ctx->status), kSmallBytes))) rc = MAASO_E_NOMEM;
  // the workspace is sized here, once: compute calls never allocate
  if (rc == MAASO_OK) rc = alloc_workspace(ctx, (size_t)MAASO_DEFAULT_WORKSPACE_BYTES);
  if (rc == MAASO_OK && !hip_ok(hipEventCreateWithFlags(&ctx->order_ev, hipEventDisableTiming))) rc = MAASO_E_HIP;
  if (rc == MAASO_OK) {
    if (!hip_ok(hipMemcpy(ctx->tab, host, (size_t)3 * cells * 4, hipMemcpyHostToDevice)) ||
        !hip_ok(hipMemset(ctx->status, 0, kSmallBytes)))
      rc = MAASO_E_HIP;
    ctx->has_degree = d->tp_degree != nullptr;
    if (rc == MAASO_OK && ctx->has_degree &&
        !hip_ok(hipMemcpy(ctx->tab + (size_t)3 * cells, d->tp_degree, (size_t)d->n_tp * 4,
                          hipMemcpyHostToDevice)))
      rc = MAASO_E_HIP;
  }
  std::free(host);
  if (rc != MAASO_OK) {
    if (ctx->order_ev) (void)hipEventDestroy(ctx->order_ev);
    if (ctx->ws) (void)hipFree(ctx->ws);
    if (ctx->tab) (void)hipFree(ctx->tab);
    if (ctx->status) (void)hipFree(ctx->status);
    (void)hipGetLastError();
    delete ctx;
    return rc;
  }
  *out_ctx = ctx;
  return MAASO_OK;
}

void maaso_ctx_destroy(maaso_ctx* ctx) {
  if (!ctx) return;
  DeviceGuard guard(ctx->device);
  (void)hipDeviceSynchronize();
  for (uint32_t i = 0; i < kMaxTimed; ++i) {
    if (ctx->ev_start[i]) (void)hipEventDestroy(ctx->ev_start[i]);
    if (ctx->ev_stop[i]) (void)hipEventDestroy(ctx->ev_stop[i]);
  }
  if (ctx->order_ev) (void)hipEventDestroy(ctx->order_ev);
  if (ctx->ws) (void)hipFree(ctx->ws);
  if (ctx->tab) (void)hipFree(ctx->tab);
  if (ctx->status) (void)hipFree(ctx->status);
  (void)hipGetLastError();
  delete ctx;
}

int maaso_ctx_device_status(maaso_ctx* ctx, uint32_t* bits) {
  if (bits) *bits = 0;
  if (!ctx) return MAASO_E_INVALID_ARG;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  uint32_t v = 0;
  if (!hip_ok(hipDeviceSynchronize())) return MAASO_E_HIP;
  if (!hip_ok(hipMemcpy(&v, ctx->status, 4, hipMemcpyDeviceToHost))) return MAASO_E_HIP;
  if (v != 0 && !hip_ok(hipMemset(ctx->status, 0, 4))) return MAASO_E_HIP;
  if (bits) *bits = v;
  if (v & MAASO_DEV_WAIT_TIMEOUT) return MAASO_E_TIMEOUT;
  return v ? MAASO_E_INVALID_ARG : MAASO_OK;
}

int maaso_ctx_set_launch_shape(maaso_ctx* ctx, uint32_t sweep_requests_per_lane,
                               uint32_t sweep_group, uint32_t sweep_blocks_per_queue,
                               uint32_t window_blocks) {
  if (!ctx) return MAASO_E_INVALID_ARG;
  const uint32_t q = sweep_requests_per_lane;
  if (q != 0 && q != 2 && q != 4 && q != 8 && q != 16) return MAASO_E_INVALID_ARG;
  ctx->sweep_q = q;
  ctx->sweep_group = sweep_group;
  ctx->sweep_blocks_per_queue = sweep_blocks_per_queue;
  ctx->window_blocks = window_blocks;
  return MAASO_OK;
}

int maaso_ctx_reserve(maaso_ctx* ctx, uint32_t max_cand, uint32_t i_pad, uint32_t max_req) {
  if (!ctx) return MAASO_E_INVALID_ARG;
  if (i_pad == 0 || i_pad > MAASO_MAX_INSTANCES || max_req > MAASO_MAX_REQUESTS) return MAASO_E_SHAPE;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  int idle = 0;
  if (!ctx->in_call.compare_exchange_strong(idle, 1, std::memory_order_acquire)) return MAASO_E_BUSY;
  const int rc = alloc_workspace(ctx, workspace_bound(ctx, max_cand ? max_cand : 1u, i_pad, max_req));
  ctx->in_call.store(0, std::memory_order_release);
  return rc;
}

int maaso_ctx_workspace(maaso_ctx* ctx, uint64_t* bytes, uint32_t* allocations) {
  if (!ctx) return MAASO_E_INVALID_ARG;
  if (bytes) *bytes = ctx->ws_bytes;
  if (allocations) *allocations = ctx->ws_allocations;
  return MAASO_OK;
}

int maaso_placement_sweep(maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                          const maaso_params* prm, uint32_t* sat_count, float* sat_ratio,
                          uint32_t* best_cand, void* hip_stream) {
  return placement_sweep_impl(ctx, pl, rq, prm, sat_count, sat_ratio, best_cand, hip_stream, false);
}

int maaso_placement_sweep_noalloc(maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                                  const maaso_params* prm, uint32_t* sat_count, float* sat_ratio,
                                  uint32_t* best_cand, void* hip_stream) {
  return placement_sweep_impl(ctx, pl, rq, prm, sat_count, sat_ratio, best_cand, hip_stream, true);
}

}  // extern "C"

namespace {

// static_scratch: the static sweep works in the library's static device array instead of the
// context's workspace and refuses what does not fit; nothing is allocated on that path.
int placement_sweep_impl(maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                         const maaso_params* prm, uint32_t* sat_count, float* sat_ratio,
                         uint32_t* best_cand, void* hip_stream, bool static_scratch) {
  int rc = check_common(ctx, pl, rq, prm);
  if (rc != MAASO_OK) return rc;
  if (!sat_count) return MAASO_E_INVALID_ARG;
  if (prm->window != 0u && rq->n_req != 0 && !rq->arrival_ticks) return MAASO_E_INVALID_ARG;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;

  const uint32_t C = pl->n_cand, I = pl->i_pad, R = rq->n_req;

  if (prm->window != 0u && R != 0) {
    // Capacity-aware form: a wavefront, or a block, walks a candidate through the request windows on its own state copy.
    SweepWindowArgs a;
    fill_sweep_window_args(a, ctx, pl, prm);
    add_sweep_window_set(a, rq, prm, sat_count, nullptr);
    {
      TimedRegion timed(ctx, s);
      rc = launch_sweep_window<false>(a, prm->policy, ctx, !static_scratch, s);
      if (rc != MAASO_OK) return rc;
    }
    hipLaunchKernelGGL(sweep_finalize_kernel, dim3(1), dim3(1024), 0, s, sat_count, C, R, sat_ratio,
                       best_cand);
    if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
    ctx->last_evaluated = nullptr;
    return MAASO_OK;
  }

  size_t bytes = 0;
  rc = static_sweep_bytes(ctx, C, I, R, bytes);
  if (rc != MAASO_OK) return rc;
  if (static_scratch) {
    if (!ctx->scratch_ptr) return MAASO_E_HIP;
    if (bytes > (size_t)MAASO_NOALLOC_SCRATCH_BYTES) return MAASO_E_SHAPE;
    return launch_static_sweep(ctx, pl, rq, prm, ctx->scratch_ptr, (size_t)MAASO_NOALLOC_SCRATCH_BYTES, sat_count, sat_ratio,
                               best_cand, s);
  }
  rc = need_workspace(ctx, bytes);
  if (rc != MAASO_OK) return rc;
  return launch_static_sweep(ctx, pl, rq, prm, ctx->ws, ctx->ws_bytes, sat_count, sat_ratio, best_cand, s);
}

}  // namespace

extern "C" {

int maaso_placement_score(maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                          const maaso_params* prm, const maaso_score_weights* wts,
                          const maaso_score_out* out, void* hip_stream) {
  return maaso_placement_score_sets(ctx, pl, 1u, rq, prm, wts, out, hip_stream);
}

int maaso_placement_score_sets(maaso_ctx* ctx, const maaso_placements* pl, uint32_t n_sets,
                               const maaso_requests* rq, const maaso_params* prm,
                               const maaso_score_weights* wts, const maaso_score_out* out,
                               void* hip_stream) {
  if (!rq || !out || n_sets == 0u || n_sets > MAASO_MAX_REQUEST_SETS) return MAASO_E_INVALID_ARG;
  ScoreSet sets[MAASO_MAX_REQUEST_SETS];
  for (uint32_t k = 0; k < n_sets; ++k) sets[k] = ScoreSet{&rq[k], &out[k], nullptr, 0u};
  const int rc = check_score_sets(ctx, pl, n_sets, sets, prm, wts);
  if (rc != MAASO_OK) return rc;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;
  return launch_score_sets(ctx, pl, n_sets, sets, prm, wts, s);
}

int maaso_profile_fit(int device, uint32_t n_tp, const uint32_t* offsets, const float* level,
                      const float* thr, uint32_t b_cap, float eps_lo, float eps_hi, double* params,
                      float* tbt) {
  if (!offsets || !level || !thr || !params || !tbt) return MAASO_E_INVALID_ARG;
  if (n_tp == 0 || b_cap == 0 || !(eps_lo > 0.0f) || !(eps_hi > eps_lo) || !std::isfinite(eps_hi))
    return MAASO_E_INVALID_ARG;
  if ((uint64_t)n_tp * ((uint64_t)b_cap + 1u) > MAASO_MAX_TABLE_CELLS) return MAASO_E_SHAPE;
  for (uint32_t t = 0; t < n_tp; ++t)
    if (offsets[t] > offsets[t + 1]) return MAASO_E_INVALID_ARG;
  const size_t n_samples = offsets[n_tp];
  for (size_t i = offsets[0]; i < n_samples; ++i)
    if (!(level[i] >= 1.0f) || !std::isfinite(level[i]) || !(thr[i] > 0.0f) || !std::isfinite(thr[i]))
      return MAASO_E_TABLE;
  int n_dev = 0;
  if (!hip_ok(hipGetDeviceCount(&n_dev)) || device < 0 || device >= n_dev) return MAASO_E_HIP;
  DeviceGuard guard(device);
  if (!guard.ok) return MAASO_E_HIP;
  // one device block: offsets | level | thr | params | tbt | flag
  const size_t cells = (size_t)n_tp * (b_cap + 1u);
  const size_t b_off = 0, b_par = (((size_t)n_tp + 1u) * 4u + 7u) & ~(size_t)7u;
  const size_t b_lvl = b_par + (size_t)n_tp * 4u * sizeof(double);
  const size_t b_thr = b_lvl + (n_samples ? n_samples : 1u) * 4u;
  const size_t b_tbt = b_thr + (n_samples ? n_samples : 1u) * 4u;
  const size_t b_bad = b_tbt + cells * 4u;
  unsigned char* dev = nullptr;
  if (!hip_ok(hipMalloc(reinterpret_cast<void**>(&dev), b_bad + 4u))) return MAASO_E_NOMEM;
  int rc = MAASO_OK;
  uint32_t bad = 0;
  if (!hip_ok(hipMemcpy(dev + b_off, offsets, ((size_t)n_tp + 1u) * 4u, hipMemcpyHostToDevice)) ||
      (n_samples && !hip_ok(hipMemcpy(dev + b_lvl, level, n_samples * 4u, hipMemcpyHostToDevice))) ||
      (n_samples && !hip_ok(hipMemcpy(dev + b_thr, thr, n_samples * 4u, hipMemcpyHostToDevice))) ||
      !hip_ok(hipMemset(dev + b_bad, 0, 4u)))
    rc = MAASO_E_HIP;
  if (rc == MAASO_OK) {
    FitArgs a;
    a.offsets = reinterpret_cast<const uint32_t*>(dev + b_off);
    a.level = reinterpret_cast<const float*>(dev + b_lvl);
    a.thr = reinterpret_cast<const float*>(dev + b_thr);
    a.b_cap = b_cap;
    a.log_eps_lo = std::log((double)eps_lo);
    a.log_eps_hi = std::log((double)eps_hi);
    a.params = reinterpret_cast<double*>(dev + b_par);
    a.tbt = reinterpret_cast<float*>(dev + b_tbt);
    a.bad = reinterpret_cast<uint32_t*>(dev + b_bad);
    hipLaunchKernelGGL(profile_fit_kernel, dim3(n_tp), dim3(kFitGrid), 0, nullptr, a);
    if (!hip_ok(hipGetLastError()) ||
        !hip_ok(hipMemcpy(params, dev + b_par, (size_t)n_tp * 4u * sizeof(double), hipMemcpyDeviceToHost)) ||
        !hip_ok(hipMemcpy(tbt, dev + b_tbt, cells * 4u, hipMemcpyDeviceToHost)) ||
        !hip_ok(hipMemcpy(&bad, dev + b_bad, 4u, hipMemcpyDeviceToHost)))
      rc = MAASO_E_HIP;
  }
  (void)hipFree(dev);
  if (rc == MAASO_OK && bad) rc = MAASO_E_TABLE;
  return rc;
}

int maaso_probe_valu(int device, uint32_t pattern, uint32_t trips, double* lane_ops_per_s,
                     uint32_t* instructions_per_trip) {
  static const uint32_t per_trip[5] = {24u, 40u, 96u, 16u, 8u};
  if (pattern > 4u || trips == 0u || !lane_ops_per_s) return MAASO_E_INVALID_ARG;
  int n_dev = 0;
  if (!hip_ok(hipGetDeviceCount(&n_dev)) || device < 0 || device >= n_dev) return MAASO_E_HIP;
  DeviceGuard guard(device);
  if (!guard.ok) return MAASO_E_HIP;
  hipDeviceProp_t prop;
  if (!hip_ok(hipGetDeviceProperties(&prop, device))) return MAASO_E_HIP;
  const uint32_t blocks = 8u * (uint32_t)(prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256);
  float* out = nullptr;
  if (!hip_ok(hipMalloc(reinterpret_cast<void**>(&out), (size_t)blocks * kProbeThreads * sizeof(float))))
    return MAASO_E_NOMEM;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = MAASO_OK;
  if (!hip_ok(hipEventCreate(&e0)) || !hip_ok(hipEventCreate(&e1))) rc = MAASO_E_HIP;
  float ms = 0.0f;
  for (int pass = 0; pass < 3 && rc == MAASO_OK; ++pass) {  // the first passes let the clock rise; the last is reported
    if (!hip_ok(hipEventRecord(e0, nullptr))) { rc = MAASO_E_HIP; break; }
    const dim3 g(blocks), b(kProbeThreads);
    switch (pattern) {
      case 0: hipLaunchKernelGGL(valu_probe_kernel<0>, g, b, 0, nullptr, out, trips, 1.0f); break;
      case 1: hipLaunchKernelGGL(valu_probe_kernel<1>, g, b, 0, nullptr, out, trips, 1.0f); break;
      case 2: hipLaunchKernelGGL(valu_probe_kernel<2>, g, b, 0, nullptr, out, trips, 1.0f); break;
      case 3: hipLaunchKernelGGL(valu_probe_kernel<3>, g, b, 0, nullptr, out, trips, 1.0f); break;
      default: hipLaunchKernelGGL(valu_probe_kernel<4>, g, b, 0, nullptr, out, trips, 1.0f); break;
    }
    if (!hip_ok(hipGetLastError()) || !hip_ok(hipEventRecord(e1, nullptr)) ||
        !hip_ok(hipEventSynchronize(e1)) || !hip_ok(hipEventElapsedTime(&ms, e0, e1)))
      rc = MAASO_E_HIP;
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  (void)hipFree(out);
  if (rc != MAASO_OK) return rc;
  if (instructions_per_trip) *instructions_per_trip = per_trip[pattern];
  *lane_ops_per_s = (double)blocks * kProbeThreads * (double)trips * per_trip[pattern] / ((double)ms * 1e-3);
  return MAASO_OK;
}

int maaso_split_by_slo(maaso_ctx* ctx, const maaso_requests* rq, uint32_t tight_classes,
                       uint32_t* prompt_len_out, uint32_t* out_len_out, uint8_t* slo_class_out,
                       uint32_t* arrival_ticks_out, uint32_t* n_tight, void* hip_stream) {
  int rc = check_split(ctx, rq, prompt_len_out, out_len_out, slo_class_out, arrival_ticks_out, n_tight);
  if (rc != MAASO_OK) return rc;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;
  return launch_split(ctx, rq, tight_classes, prompt_len_out, out_len_out, slo_class_out,
                      arrival_ticks_out, n_tight, s);
}

int maaso_ins_deploy_select(maaso_ctx* ctx, const maaso_placements* pl, const float* score,
                            const uint32_t* chain_offsets, uint32_t n_chains, uint32_t n_gpus,
                            float* phi_star, int32_t* cand_star, void* hip_stream) {
  const int rc = check_select(ctx, pl, score, n_gpus, phi_star, cand_star);
  if (rc != MAASO_OK) return rc;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;
  return launch_select(ctx, pl, 1u, &score, chain_offsets, n_chains, n_gpus, &phi_star, &cand_star, s);
}

int maaso_resource_partition(maaso_ctx* ctx, uint32_t n_gpus, const float* phi_t_star,
                             const float* phi_l_star, const float* phi_h_star,
                             const int32_t* cand_t_star, const int32_t* cand_l_star,
                             const int32_t* cand_h_star, uint64_t n_req_l, uint64_t n_req,
                             uint32_t* partition, float* phi_opt, void* hip_stream) {
  if (!ctx || !phi_t_star || !phi_l_star || !partition || !phi_opt) return MAASO_E_INVALID_ARG;
  if (n_req_l > n_req) return MAASO_E_INVALID_ARG;
  if (n_gpus > MAASO_MAX_GPUS) return MAASO_E_SHAPE;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;
  PartitionArgs a;
  a.n_gpus = n_gpus;
  // initial share of the relaxed sub-cluster: floor(|R_l| / |R| * |G|), from the exact quotient
  a.g_l_cap = n_req == 0 ? 0u : (uint32_t)(((unsigned __int128)n_req_l * n_gpus) / n_req);
  a.n_tight = nullptr;
  a.n_req = 0u;
  a.phi_t_star = phi_t_star;
  a.phi_l_star = phi_l_star;
  a.phi_h_star = phi_h_star;
  a.cand_t_star = cand_t_star;
  a.cand_l_star = cand_l_star;
  a.cand_h_star = cand_h_star;
  a.out = partition;
  a.phi_opt = phi_opt;
  hipLaunchKernelGGL(resource_partition_kernel, dim3(1), dim3(kPartitionThreads), 0, s, a);
  return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
}

int maaso_batch_size_prune(maaso_ctx* ctx, uint32_t n_cand, const uint32_t* group_offsets,
                           uint32_t n_groups, const uint32_t* sat_count, const float* latency,
                           uint8_t* keep, uint32_t* n_kept, void* hip_stream) {
  if (!ctx || !group_offsets || !n_kept) return MAASO_E_INVALID_ARG;
  if (n_cand != 0u && (!sat_count || !latency || !keep)) return MAASO_E_INVALID_ARG;
  if (n_groups > 0x7fffffffu) return MAASO_E_SHAPE;
  if (n_groups == 0u) return MAASO_OK;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;
  PruneArgs a;
  a.n_cand = n_cand;
  a.group_offsets = group_offsets;
  a.n_groups = n_groups;
  a.sat_count = sat_count;
  a.latency = latency;
  a.keep = keep;
  a.n_kept = n_kept;
  a.status = ctx->status;
  const bool small = prune_in_fours(n_cand, n_groups);
  if (small) hipLaunchKernelGGL(batch_prune_small_kernel, dim3(n_groups / 4u + (n_groups % 4u != 0u ? 1u : 0u)), dim3(kPruneTile), 0, s, a);
  else if (n_groups <= kPruneSingle) hipLaunchKernelGGL((batch_prune_kernel<true>), dim3(n_groups), dim3(kPruneTile), 0, s, a);
  else hipLaunchKernelGGL((batch_prune_kernel<false>), dim3(n_groups), dim3(kPruneTile), 0, s, a);
  if (n_groups > (small ? kPruneLook : kPruneSingle)) {
    const uint32_t per_block = std::max(8u * (uint32_t)kPruneTile, (uint32_t)(((uint64_t)n_groups + 1023u) / 1024u));
    hipLaunchKernelGGL(prune_overlaps_kernel, dim3((uint32_t)(((uint64_t)n_groups + per_block - 1u) / per_block)), dim3(kPruneTile), 0, s, a,
                       per_block);
  }
  return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
}

int maaso_resource_partition_requests(maaso_ctx* ctx, const maaso_placements* pl,
                                      const uint32_t* chain_offsets, uint32_t n_chains,
                                      uint32_t n_gpus, const maaso_requests* rq,
                                      uint32_t tight_classes, const maaso_params* prm,
                                      const maaso_score_weights* wts,
                                      const maaso_partition_work* wk, void* hip_stream) {
  if (!wk || !rq) return MAASO_E_INVALID_ARG;
  if (!wk->score_t || !wk->score_l || !wk->sat_t || !wk->sat_l || !wk->phi_t_star ||
      !wk->phi_l_star || !wk->cand_t_star || !wk->cand_l_star || !wk->partition || !wk->phi_opt)
    return MAASO_E_INVALID_ARG;
  const bool homogeneous = wk->score_h != nullptr;
  if (homogeneous && (!wk->sat_h || !wk->phi_h_star || !wk->cand_h_star)) return MAASO_E_INVALID_ARG;
  int rc = check_split(ctx, rq, wk->prompt_len_split, wk->out_len_split, wk->slo_class_split,
                       wk->arrival_ticks_split, wk->n_tight);
  if (rc != MAASO_OK) return rc;
  // the split arrays as one request set of n_req requests; its two sides are cut on the device
  maaso_requests whole = *rq;
  whole.prompt_len = wk->prompt_len_split;
  whole.out_len = wk->out_len_split;
  whole.slo_class = wk->slo_class_split;
  whole.arrival_ticks = rq->arrival_ticks ? wk->arrival_ticks_split : nullptr;
  const maaso_score_out out_t = {wk->sat_t, nullptr, nullptr, nullptr, wk->score_t, nullptr};
  const maaso_score_out out_l = {wk->sat_l, nullptr, nullptr, nullptr, wk->score_l, nullptr};
  const maaso_score_out out_h = {wk->sat_h, nullptr, nullptr, nullptr, wk->score_h, nullptr};
  ScoreSet sets[3];
  uint32_t n_sets = 0;
  if (homogeneous) sets[n_sets++] = ScoreSet{rq, &out_h, nullptr, 0u};
  sets[n_sets++] = ScoreSet{&whole, &out_t, wk->n_tight, 1u};
  sets[n_sets++] = ScoreSet{&whole, &out_l, wk->n_tight, 2u};
  rc = check_score_sets(ctx, pl, n_sets, sets, prm, wts);
  if (rc != MAASO_OK) return rc;
  rc = check_select(ctx, pl, wk->score_t, n_gpus, wk->phi_t_star, wk->cand_t_star);
  if (rc != MAASO_OK) return rc;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;
  rc = launch_split(ctx, rq, tight_classes, wk->prompt_len_split, wk->out_len_split,
                    wk->slo_class_split, wk->arrival_ticks_split, wk->n_tight, s);
  if (rc != MAASO_OK) return rc;
  rc = launch_score_sets(ctx, pl, n_sets, sets, prm, wts, s);
  if (rc != MAASO_OK) return rc;
  {
    const float* scores[3] = {wk->score_t, wk->score_l, wk->score_h};
    float* phis[3] = {wk->phi_t_star, wk->phi_l_star, wk->phi_h_star};
    int32_t* cands[3] = {wk->cand_t_star, wk->cand_l_star, wk->cand_h_star};
    rc = launch_select(ctx, pl, homogeneous ? 3u : 2u, scores, chain_offsets, n_chains, n_gpus, phis,
                       cands, s);
  }
  if (rc != MAASO_OK) return rc;
  PartitionArgs a;
  a.n_gpus = n_gpus;
  a.g_l_cap = 0u;
  a.n_tight = wk->n_tight;  // G'_l = floor(|R_l| * |G| / |R|) from the device's |R_t|
  a.n_req = rq->n_req;
  a.phi_t_star = wk->phi_t_star;
  a.phi_l_star = wk->phi_l_star;
  a.phi_h_star = homogeneous ? wk->phi_h_star : nullptr;
  a.cand_t_star = wk->cand_t_star;
  a.cand_l_star = wk->cand_l_star;
  a.cand_h_star = homogeneous ? wk->cand_h_star : nullptr;
  a.out = wk->partition;
  a.phi_opt = wk->phi_opt;
  hipLaunchKernelGGL(resource_partition_kernel, dim3(1), dim3(kPartitionThreads), 0, s, a);
  return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
}

int maaso_score_assign(maaso_ctx* ctx, const maaso_placements* pl, const maaso_requests* rq,
                       const maaso_params* prm, const maaso_assign_out* out, void* hip_stream) {
  if (pl && pl->n_cand != 1u) return MAASO_E_INVALID_ARG;
  return score_assign_impl(ctx, pl, nullptr, rq, prm, out, hip_stream);
}

int maaso_score_assign_selected(maaso_ctx* ctx, const maaso_placements* pl, const uint32_t* cand,
                                const maaso_requests* rq, const maaso_params* prm,
                                const maaso_assign_out* out, void* hip_stream) {
  if (!cand) return MAASO_E_INVALID_ARG;
  return score_assign_impl(ctx, pl, cand, rq, prm, out, hip_stream);
}

}  // extern "C"

namespace {

// The windowed distributor in launches over the requests laid out, as many windows at a time as the workspace
// takes.  kNotTaken, nothing launched, where that are too few.
constexpr int kNotTaken = 1;
int launch_assign_ordered(maaso_ctx* ctx, const AssignArgs& a, const maaso_placements* pl, const maaso_requests* rq,
                          const maaso_params* prm, const maaso_assign_out* out, bool lat, hipStream_t s) {
  const uint32_t R = rq->n_req, I = pl->i_pad, size_log2 = 6;
  SweepWindowSet set{};
  set.n_req = R;
  set.window = prm->window;
  const uint64_t n_windows = ((uint64_t)R + prm->window - 1u) / prm->window;
  // of one window; the arrays' starts are rounded up
  unsigned char* at = nullptr;
  const OrderedSet one = plan_set(set, a.n_slo, size_log2, 1u, at);
  const uint64_t places = (uint64_t)one.batches << size_log2;
  const uint64_t per_window = places * 8u + (uint64_t)one.batches * sizeof(Batch) + 4u + (uint64_t)I * 20u;
  // A captured one leaves a quarter of the workspace to the requests of windowed sweeps, which keep out of what it uses.
  const uint64_t held = is_captured(s) ? ctx->ws_bytes / 4u * 3u : ctx->ws_bytes;
  const uint64_t room = held > 8192u ? held - 8192u : 0u;
  uint64_t at_once = std::min(room / per_window, n_windows);
  at_once = std::min(at_once, (uint64_t)(1u << 24) / one.segments);
  if (at_once == 0u || (at_once < n_windows && at_once < 64u)) return kNotTaken;
  auto al = [](const void* p, uintptr_t m) { return (reinterpret_cast<uintptr_t>(p) & m) == 0; };
  const bool vec = prm->window % 4u == 0u && al(rq->prompt_len, 15) && al(rq->out_len, 15) && al(rq->slo_class, 3) &&
                   al(out->chosen, 15) && al(out->slack, 15) && al(out->ttft, 15) && al(out->tbt, 15) && al(out->e2e, 15);
  const uint32_t window = std::min(prm->window, R);
  const uint32_t per_pass = kAssignThreads * (vec ? 4u : 1u);
  const uint32_t per_block = std::min((window + per_pass - 1u) / per_pass, 4u) * per_pass;
  const uint32_t per_window_blocks = (window + per_block - 1u) / per_block;
  if ((uint64_t)per_window_blocks * at_once > 0x7fffffffull) return kNotTaken;
  const uint32_t segment = std::min(window, kSegment);
  use_workspace(ctx, 8192u + at_once * per_window, s);
  TimedRegion timed(ctx, s);
  for (uint64_t w0 = 0; w0 < n_windows; w0 += at_once) {
    const uint32_t count = (uint32_t)std::min(at_once, n_windows - w0);
    const size_t skip = (size_t)w0 * prm->window;
    OrderArgs o;
    o.n_slo = a.n_slo;
    o.status = a.status;
    o.n_sets = 1u;
    o.first[0] = 0u;
    SweepWindowSet& t = o.sets[0];
    t = SweepWindowSet{};
    t.n_req = (uint32_t)(R - skip);
    t.window = prm->window;
    t.prompt_len = rq->prompt_len + skip;
    t.out_len = rq->out_len + skip;
    t.slo_class = rq->slo_class + skip;
    t.arrival_ticks = rq->arrival_ticks + skip;
    at = static_cast<unsigned char*>(ctx->ws);
    SweepWindowSet whole = t;
    whole.n_req = R;  // (windows of one size, also where the rest is shorter than one)
    o.to[0] = plan_set(whole, a.n_slo, size_log2, count, at);
    StateRun run;
    run.n_req = R;
    run.window = prm->window;
    run.w0 = (uint32_t)w0;
    run.n_windows = count;
    run.recs = reinterpret_cast<float4*>(at);
    at += up256((size_t)count * I * sizeof(float4));
    run.occ = reinterpret_cast<int32_t*>(at);
    hipLaunchKernelGGL(order_requests_kernel, dim3(count * o.to[0].segments), dim3(segment <= 256u * kOrderPer ? 256u : 1024u),
                       order_lds(segment, a.n_slo, 1u << size_log2), s, o);
    const size_t lds = (size_t)3 * ctx->cells * sizeof(float);
    auto states = [&](auto s_, auto sq_) {
      hipLaunchKernelGGL((assign_states_kernel<s_(), 4, sq_()>), dim3(1), dim3(5 * 64), lds, s, a, o.to[0], run);
    };
    auto states_by_slots = [&](auto sq_) {
      if (I <= 64u) states(std::integral_constant<int, 1>{}, sq_);
      else if (I <= 128u) states(std::integral_constant<int, 2>{}, sq_);
      else states(std::integral_constant<int, 4>{}, sq_);
    };
    if (prm->policy) states_by_slots(std::true_type{});
    else states_by_slots(std::false_type{});
    if (a.chosen || a.slack || lat) {
      const int list = I <= 16u && !prm->policy ? 0 : I <= 64u ? 1 : I <= 128u ? 2 : 4;
      const dim3 g(count * per_window_blocks), b(kAssignThreads);
      auto launch = [&](auto lat_, auto v_, auto sq_, auto list_) {
        hipLaunchKernelGGL((assign_recorded_kernel<lat_(), v_(), sq_(), list_()>), g, b, 0, s, a, run, per_window_blocks, per_block);
      };
      auto by_list = [&](auto lat_, auto v_, auto sq_) {
        if (list == 0) launch(lat_, v_, std::false_type{}, std::integral_constant<int, 0>{});
        else if (list == 1) launch(lat_, v_, sq_, std::integral_constant<int, 1>{});
        else if (list == 2) launch(lat_, v_, sq_, std::integral_constant<int, 2>{});
        else launch(lat_, v_, sq_, std::integral_constant<int, 4>{});
      };
      auto by_policy = [&](auto lat_, auto v_) {
        if (prm->policy) by_list(lat_, v_, std::true_type{});
        else by_list(lat_, v_, std::false_type{});
      };
      auto by_width = [&](auto lat_) {
        if (vec) by_policy(lat_, std::integral_constant<int, 4>{});
        else by_policy(lat_, std::integral_constant<int, 1>{});
      };
      if (lat) by_width(std::true_type{});
      else by_width(std::false_type{});
    }
    if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
  }
  return MAASO_OK;
}

int score_assign_impl(maaso_ctx* ctx, const maaso_placements* pl, const uint32_t* cand_sel,
                      const maaso_requests* rq, const maaso_params* prm, const maaso_assign_out* out,
                      void* hip_stream) {
  int rc = check_common(ctx, pl, rq, prm);
  if (rc != MAASO_OK) return rc;
  if (!out || (!out->chosen && !out->n_satisfied)) return MAASO_E_INVALID_ARG;
  const uint32_t R = rq->n_req;
  if (prm->window != 0u && R != 0 && !rq->arrival_ticks) return MAASO_E_INVALID_ARG;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  CallGuard call(ctx, s);
  if (call.rc != MAASO_OK) return call.rc;

  AssignArgs a;
  fill_assign_args(a, ctx, pl, rq, prm, out);
  a.cand_sel = cand_sel;
  const bool lat = out->ttft || out->tbt || out->e2e;
  if (R == 0) {
    hipLaunchKernelGGL(assign_init_kernel, dim3(1), dim3(64), 0, s, a.n_satisfied);
    return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
  }
  if (prm->window == 0u) {
    // 16-byte accesses, four requests per thread, when every array allows it
    auto al = [](const void* p, uintptr_t m) { return (reinterpret_cast<uintptr_t>(p) & m) == 0; };
    const bool vec = al(rq->prompt_len, 15) && al(rq->out_len, 15) && al(rq->slo_class, 3) &&
                     al(out->chosen, 15) && al(out->slack, 15) && al(out->ttft, 15) &&
                     al(out->tbt, 15) && al(out->e2e, 15);
    const uint32_t per_block = kAssignThreads * (vec ? 4u : 1u);
    uint32_t blocks = (uint32_t)(((uint64_t)R + per_block - 1) / per_block);
    // few instance slots: records live in registers and the loop needs no LDS (HBM-bound shape)
    const bool few = pl->i_pad <= 8u;
    // persistent blocks; measured on the HBM-bound shape: 3 per compute unit (all resident, 213 us)
    // beat 2 (228), 4 (219), 5 (254) and 8 (222)
    const uint32_t cap = (uint32_t)ctx->n_cu * (few ? 3u : 8u);
    if (blocks > cap) blocks = cap;
    TimedRegion timed(ctx, s);
    // How wide the listing of instances gets, and where comparing all of them is quicker: few slots, and a part of
    // the threads with a second group of requests.  Measured, all / listed, largest slack, jittered profiles: 9
    // slots, 1,500,000 requests (one group): 11.5 / 10.4 us; 2,500,000 (one or two): 15.6 / 18.0; 5,000,000: 25.1 / 22.6; 12
    // slots: 12.7 / 10.2, 16.9 / 19.5, - / 22.6; 16 slots: 14.2 / 10.7, 19.4 / 19.9.  Shortest queue, 9 slots: 16.9 / 12.0, 21.2 / 18.9.
    const uint64_t n_vec = (uint64_t)R / (vec ? 4u : 1u), stride = (uint64_t)blocks * kAssignThreads;
    const bool all = !prm->policy && pl->i_pad <= 16u && n_vec > stride && n_vec <= 2u * stride;
    const int list = few || all ? 0 : pl->i_pad <= 64u ? 1 : pl->i_pad <= 128u ? 2 : 4;
    auto launch = [&](auto lat_, auto v_, auto nreg_, auto sq_, auto list_) {
      hipLaunchKernelGGL((assign_static_kernel<lat_(), v_(), nreg_(), sq_(), list_()>), dim3(blocks), dim3(kAssignThreads), 0, s, a);
    };
    auto by_list = [&](auto lat_, auto v_, auto sq_) {
      if (few) launch(lat_, v_, std::integral_constant<int, 8>{}, sq_, std::integral_constant<int, 0>{});
      else if (list == 0) launch(lat_, v_, std::integral_constant<int, 0>{}, std::false_type{}, std::integral_constant<int, 0>{});
      else if (list == 1) launch(lat_, v_, std::integral_constant<int, 0>{}, sq_, std::integral_constant<int, 1>{});
      else if (list == 2) launch(lat_, v_, std::integral_constant<int, 0>{}, sq_, std::integral_constant<int, 2>{});
      else launch(lat_, v_, std::integral_constant<int, 0>{}, sq_, std::integral_constant<int, 4>{});
    };
    auto by_policy = [&](auto lat_, auto v_) {
      if (prm->policy) by_list(lat_, v_, std::true_type{});
      else by_list(lat_, v_, std::false_type{});
    };
    auto by_width = [&](auto lat_) {
      if (vec) by_policy(lat_, std::integral_constant<int, 4>{});
      else by_policy(lat_, std::integral_constant<int, 1>{});
    };
    if (lat) by_width(std::true_type{});
    else by_width(std::false_type{});
    return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
  }

  // Short windows (down to one request per window, the online distributor taken literally): one
  // wavefront with the instances in its lanes and no device-wide barrier.
  // The window_blocks knob set to a value asks for the persistent kernel below whatever the window, and so does
  // its profile for the windows that it describes.
  const uint32_t short_window = assign_short_window(pl->i_pad, a.bounds.narrow_queue);
  const bool profiled = ctx->window_profile && prm->window > (pl->i_pad <= 128u ? 4u : 2u);
  if (prm->policy == 0u && prm->window <= short_window && ctx->window_blocks == 0u && !profiled) {
    const size_t lds = ((size_t)ctx->cells + 1u) * sizeof(float4);
    TimedRegion timed(ctx, s);
    auto launch = [&](auto lat_, auto s_, auto fits_) {
      hipLaunchKernelGGL((assign_seq_kernel<lat_(), s_(), fits_()>), dim3(1), dim3(64), lds, s, a, prm->window);
    };
    auto by_form = [&](auto lat_, auto s_) {
      if (a.bounds.narrow_queue) launch(lat_, s_, std::true_type{});
      else launch(lat_, s_, std::false_type{});
    };
    auto by_slots = [&](auto lat_) {
      if (pl->i_pad <= 64u) by_form(lat_, std::integral_constant<int, 1>{});
      else if (pl->i_pad <= 128u) by_form(lat_, std::integral_constant<int, 2>{});
      else by_form(lat_, std::integral_constant<int, 4>{});
    };
    if (lat) by_slots(std::true_type{});
    else by_slots(std::false_type{});
    return hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
  }

  // Few slots, or long windows: in launches over the requests laid out.  The window_blocks knob and the profile ask for
  // the persistent kernel here too.
  const bool ordered = a.bounds.narrow && assign_lays_out(pl->i_pad, prm->window < R ? prm->window : R,
                                                          ((uint64_t)R + prm->window - 1u) / prm->window, prm->policy != 0u);
  if (ordered && ctx->window_blocks == 0u && !(ctx->window_profile && !prm->policy && !lat)) {
    const int done = launch_assign_ordered(ctx, a, pl, rq, prm, out, lat, s);
    if (done != kNotTaken) {
      ctx->window_profiled = false;
      return done;
    }
  }

  // Windowed: one persistent kernel; all blocks must be resident at once (one per compute unit at
  // most).  Each request is spread over LPR lanes so that a window fills the blocks.
  rc = need_workspace(ctx, sizeof(WindowWs));
  if (rc != MAASO_OK) return rc;
  use_workspace(ctx, sizeof(WindowWs), s);
  WindowWs* ws = static_cast<WindowWs*>(ctx->ws);
  const uint32_t per_window = prm->window < R ? prm->window : R;
  // More blocks shorten a window's scoring (more lanes per request, shorter instance walks) and
  // lengthen the window boundary, where every block adds to every instance's accumulators and the
  // owners of the instances read them until all blocks are counted in.  Measured per window
  // (16 / 32 / 64 / 128 blocks): 64 instances, windows of 4096: 3.63 / 3.15 / 3.81 / 5.77 us;
  // 256 instances, 4096: 7.2 / 5.4 / 5.7 / 7.6; 64 instances, 32768: 13.0 / 8.0 / 6.2 / 6.9;
  // 256 instances, 32768: 39.9 / 22.0 / 13.5 / 11.5.  Lanes per request are then chosen so that a
  // window is scored in one pass.
  const uint64_t window_triples = (uint64_t)per_window * pl->i_pad;
  uint32_t nb = ctx->window_blocks ? ctx->window_blocks
                                   : (window_triples < (1ull << 21) ? 32u : (window_triples < (1ull << 23) ? 64u : 128u));
  if (nb > (uint32_t)ctx->n_cu) nb = (uint32_t)ctx->n_cu;
  if (nb == 0) nb = 1;
  uint32_t lpr = 1;
  while (lpr < 64u && lpr * 2u <= pl->i_pad &&
         (uint64_t)per_window * (lpr * 2u) <= (uint64_t)nb * kWindowThreads)
    lpr *= 2u;
  const uint64_t need = ((uint64_t)per_window * lpr + kWindowThreads - 1) / kWindowThreads;
  if (need < nb) nb = (uint32_t)(need ? need : 1);
  hipLaunchKernelGGL(window_init_kernel, dim3(1), dim3(256), 0, s, ws, a.n_satisfied);
  if (!hip_ok(hipGetLastError())) return MAASO_E_HIP;
  uint32_t spin = ctx->spin_limit;
  uint32_t window_v = prm->window;
  const size_t wlds = (size_t)3 * ctx->cells * sizeof(float);  // profile tables in LDS
  TimedRegion timed(ctx, s);
  // The kernel's device-wide barrier needs every block resident at once.  A cooperative launch
  // guarantees that or is refused; where the device has none, the occupancy of the kernel decides on
  // the host (and the bounded spin remains the net under other work on the device).
  void* kargs[] = {&a, &window_v, &ws, &spin};
  hipError_t launched = hipSuccess;
  auto launch = [&](const void* fn) {
    if (ctx->cooperative) {
      launched = hipLaunchCooperativeKernel(fn, dim3(nb), dim3(kWindowThreads), kargs, (unsigned)wlds, s);
    } else {
      int per_cu = 0;
      launched = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, fn, kWindowThreads, wlds);
      if (launched == hipSuccess && (uint64_t)per_cu * (uint64_t)ctx->n_cu < nb)
        launched = hipErrorCooperativeLaunchTooLarge;
      if (launched == hipSuccess)
        launched = hipLaunchKernel(fn, dim3(nb), dim3(kWindowThreads), kargs, wlds, s);
    }
  };
  ctx->window_profiled = ctx->window_profile && !prm->policy && !lat;
#define MAASO_LAUNCH_WINDOW(LPR)                                                                  \
  do {                                                                                            \
    if (prm->policy) /* latency outputs are null-checked in the kernel: one variant serves both */ \
      launch(reinterpret_cast<const void*>(&assign_window_kernel<LPR, true, true>));               \
    else if (lat)                                                                                  \
      launch(reinterpret_cast<const void*>(&assign_window_kernel<LPR, true, false>));              \
    else if (ctx->window_profiled)                                                                 \
      launch(reinterpret_cast<const void*>(&assign_window_kernel<LPR, false, false, true>));       \
    else                                                                                           \
      launch(reinterpret_cast<const void*>(&assign_window_kernel<LPR, false, false>));             \
  } while (0)
  switch (lpr) {
    case 1: MAASO_LAUNCH_WINDOW(1); break;
    case 2: MAASO_LAUNCH_WINDOW(2); break;
    case 4: MAASO_LAUNCH_WINDOW(4); break;
    case 8: MAASO_LAUNCH_WINDOW(8); break;
    case 16: MAASO_LAUNCH_WINDOW(16); break;
    case 32: MAASO_LAUNCH_WINDOW(32); break;
    default: MAASO_LAUNCH_WINDOW(64); break;
  }
#undef MAASO_LAUNCH_WINDOW
  if (launched == hipErrorCooperativeLaunchTooLarge) {
    (void)hipGetLastError();
    return MAASO_E_RESIDENCY;
  }
  return hip_ok(launched) && hip_ok(hipGetLastError()) ? MAASO_OK : MAASO_E_HIP;
}

}  // namespace

extern "C" {

int maaso_ctx_kernel_timing(maaso_ctx* ctx, int enable) {
  if (!ctx) return MAASO_E_INVALID_ARG;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  if (enable && !ctx->ev_start[0]) {
    for (uint32_t i = 0; i < kMaxTimed; ++i)
      if (!hip_ok(hipEventCreate(&ctx->ev_start[i])) || !hip_ok(hipEventCreate(&ctx->ev_stop[i])))
        return MAASO_E_HIP;
  }
  ctx->timing = enable != 0;
  ctx->n_timed = 0;
  return MAASO_OK;
}

int maaso_ctx_kernel_elapsed(maaso_ctx* ctx, float* total_ms, uint32_t* launches) {
  if (!ctx || !total_ms || !launches) return MAASO_E_INVALID_ARG;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  float sum = 0.0f;
  for (uint32_t i = 0; i < ctx->n_timed; ++i) {
    float ms = 0.0f;
    if (!hip_ok(hipEventSynchronize(ctx->ev_stop[i])) ||
        !hip_ok(hipEventElapsedTime(&ms, ctx->ev_start[i], ctx->ev_stop[i])))
      return MAASO_E_HIP;
    sum += ms;
  }
  *total_ms = sum;
  *launches = ctx->n_timed;
  ctx->n_timed = 0;
  return MAASO_OK;
}

int maaso_ctx_kernel_durations(maaso_ctx* ctx, float* durations_ms, uint32_t cap, uint32_t* launches) {
  if (!ctx || !durations_ms || !launches) return MAASO_E_INVALID_ARG;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  const uint32_t n = ctx->n_timed < cap ? ctx->n_timed : cap;
  for (uint32_t i = 0; i < n; ++i) {
    float ms = 0.0f;
    if (!hip_ok(hipEventSynchronize(ctx->ev_stop[i])) ||
        !hip_ok(hipEventElapsedTime(&ms, ctx->ev_start[i], ctx->ev_stop[i])))
      return MAASO_E_HIP;
    durations_ms[i] = ms;
  }
  *launches = n;
  ctx->n_timed = 0;
  return MAASO_OK;
}

int maaso_ctx_sweep_evaluated(maaso_ctx* ctx, uint64_t* pairs, uint64_t* pairs_without_wait) {
  if (!ctx || !pairs) return MAASO_E_INVALID_ARG;
  *pairs = 0;
  if (pairs_without_wait) *pairs_without_wait = 0;
  if (!ctx->last_evaluated) return MAASO_OK;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  unsigned long long v[2] = {0, 0};
  if (!hip_ok(hipDeviceSynchronize())) return MAASO_E_HIP;
  if (!hip_ok(hipMemcpy(v, ctx->last_evaluated, sizeof(v), hipMemcpyDeviceToHost))) return MAASO_E_HIP;
  *pairs = v[0];
  if (pairs_without_wait) *pairs_without_wait = v[1];
  return MAASO_OK;
}

int maaso_ctx_window_profile(maaso_ctx* ctx, int enable) {
  if (!ctx) return MAASO_E_INVALID_ARG;
  ctx->window_profile = enable != 0;
  ctx->window_profiled = false;
  return MAASO_OK;
}

int maaso_ctx_window_phases(maaso_ctx* ctx, uint64_t cycles[6]) {
  if (!ctx || !cycles) return MAASO_E_INVALID_ARG;
  for (int i = 0; i < 6; ++i) cycles[i] = 0;
  if (!ctx->window_profiled) return MAASO_OK;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  if (!hip_ok(hipDeviceSynchronize())) return MAASO_E_HIP;
  const WindowWs* ws = static_cast<const WindowWs*>(ctx->ws);
  unsigned long long v[6];
  if (!hip_ok(hipMemcpy(v, ws->phase, sizeof(v), hipMemcpyDeviceToHost))) return MAASO_E_HIP;
  for (int i = 0; i < 6; ++i) cycles[i] = v[i];
  return MAASO_OK;
}

int maaso_ctx_set_cooperative(maaso_ctx* ctx, int enable) {
  if (!ctx) return MAASO_E_INVALID_ARG;
  DeviceGuard guard(ctx->device);
  if (!guard.ok) return MAASO_E_HIP;
  int can = 0;
  if (enable && !hip_ok(hipDeviceGetAttribute(&can, hipDeviceAttributeCooperativeLaunch, ctx->device))) can = 0;
  ctx->cooperative = enable ? can : 0;
  return MAASO_OK;
}

int maaso_ctx_set_wait_limit(maaso_ctx* ctx, uint32_t polls) {
  if (!ctx) return MAASO_E_INVALID_ARG;
  ctx->spin_limit = polls;
  return MAASO_OK;
}

}  // extern "C"
