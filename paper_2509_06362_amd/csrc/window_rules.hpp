// Index rules of the windowed sweeps that are the same on any machine: plain C++, used by the kernels and
// tested on the CPU.
#pragma once

#include <stdint.h>

namespace maaso {

// Whether the arrival of the request behind request r is read.  Time passes only between two windows, and
// only a set that has two comes with arrivals for certain: a static score is one window over all of its
// requests and may have none (a null pointer).
constexpr bool reads_arrival_behind(uint32_t r, uint32_t n_req, uint32_t window) {
  return n_req > window && r < n_req && n_req - r > 1u;
}

// Buffers of a window's admitted sums where the wavefronts of a block share a candidate, used in turn, one
// barrier per window.  Between two barriers any wavefront may be anywhere in: reading the sums of the
// window before, adding to those of this window, clearing a buffer.  The one to clear is therefore the
// next: it was read before the last barrier, which everybody has passed, and is added to behind the
// coming one.
constexpr uint32_t kSumBuffers = 3;
constexpr uint32_t next_sum_buffer(uint32_t buf) { return buf + 1u == kSumBuffers ? 0u : buf + 1u; }
constexpr uint32_t cleared_sum_buffer(uint32_t buf) { return next_sum_buffer(buf); }

// Fewer ticks than this between two windows, and no request completes on an instance on a strategy's row w (tbt
// seconds per token), if it held at most w - 1 requests when the window opened, or w is its batch cap: a
// request completes once run * seconds reaches the service time, with run <= w - 1 + window the requests that
// run and a service time of at least s_bar * tbt (the occupancy penalty is a factor of one or more).  Ticks,
// product, service time and the quotient here are rounded once each by at most 2^-24; 2^-10 is taken off.
constexpr uint32_t row_safe_ticks(float s_bar, float tbt, uint32_t w, uint32_t window) {
  const float x = (s_bar * tbt) / ((float)w + (float)(window - 1u)) * (1048576.0f * (1.0f - 0x1p-10f));
  return x < 4e9f ? (uint32_t)x : 4000000000u;
}

// The longest windows of a windowed sweep or score that go to the kernel whose lanes are the instances while a request
// is scored (no search for the instances a request can be given, but all of them at every request).  `narrow`: queues
// fit 32 bits (AdmissionBounds::narrow_queue), so its 32-bit form runs wherever the slots allow it; else its general form.
// Measured, the lanes-are-requests kernel's time over its, least of three layouts (jittered and smooth profiles, loaded and
// fresh instances) and of 2700 and 9000 candidates:
//   32 bits: 8 slots, windows of 12: 1.13, 13: 1.08, 16: 0.92; 16 slots, 16: 1.16, 20: 0.96; 24 slots, 20: 1.08; 32 slots, 20: 1.18;
//   40 slots, 24: 1.10, 28: 0.94; 64 slots, 24: 1.18, 28: 1.02; 100 slots, 24: 1.15, 28: 0.98; 136 slots, 28: 1.03; 200 slots, 28:
//   1.05, 34: 0.88.  With the score's sums, which cost it more: 8 slots, 12: 1.14; 16 slots, 16: 1.17; 24 slots, 20: 1.12; 40 slots,
//   24: 1.09; 64 slots, 24: 1.20; 136 slots, 28: 1.01; 200 slots, 28: 1.11.
//   General (first-token deadlines of 600 s): 4 slots, 6: 1.08, 8: 0.90; 8 slots, 9: 1.03, 10: 0.94; 12 slots, 10: 1.07; 16 slots, 12:
//   1.02, 14: 0.89; 24 slots, 12: 1.11, 14: 0.98; 32 slots, 14: 1.07, 16: 0.97; 40 slots, 16: 1.01, 18: 0.92; 64 slots, 16: 1.11, 18: 0.99;
//   100 slots, 18: 1.08, 20: 0.98; 128 slots, 18: 1.11; 136 slots, 20: 1.04, 24: 0.87; 200 slots, 24: 0.97; 256 slots, 24: 1.03, 26: 0.96.
constexpr uint32_t sweep_short_window(uint32_t i_pad, bool score, bool narrow) {
  if (!narrow)
    return i_pad >= 192u ? 24u : i_pad > 128u ? 20u : i_pad >= 100u ? 18u : i_pad >= 40u ? 16u
           : i_pad >= 32u ? 14u : i_pad >= 16u ? 12u : i_pad >= 8u ? 9u : 6u;
  if (i_pad >= 40u) return i_pad > 128u ? (score ? 24u : 28u) : (score ? 20u : 24u);
  return i_pad >= 24u ? (score ? 18u : 20u) : i_pad >= 16u ? 16u : i_pad >= 8u ? 12u : 8u;
}

// The same for the distributor, one wavefront against the persistent kernel.  Measured, the persistent kernel's time
// over one wavefront's, 32 bits: windows of 5 / 8 / 10 / 12 requests: 4 slots: 1.87 / 1.28 / 1.05 / 0.91, 64: 2.01 / 1.39 / 1.17 /
// 1.02, 100: 1.60 / 1.09 / 0.93 / 0.80, 128: 1.59 / 1.08 / 0.91; of 3 / 4 / 5 / 6: 200: 1.87 / 1.52 / 1.27 / 1.09, 256: 1.67 / 1.35 / 1.15 /
// 0.99.  General: of 7 / 8 / 9: 4 slots: 1.19 / 1.08 / 0.97, 64: 1.16 / 1.04 / 0.97; of 5 / 6 / 7: 65: 1.26 / 1.08 / 0.95, 128: 1.21 /
// 1.04 / 0.92; of 4 / 5: 129: 1.16 / 0.98, 256: 1.10 / 0.94.
constexpr uint32_t assign_short_window(uint32_t i_pad, bool narrow) {
  if (!narrow) return i_pad <= 64u ? 8u : i_pad <= 128u ? 6u : 4u;
  return i_pad <= 64u ? 10u : i_pad <= 128u ? 8u : 5u;
}

// Whether the windowed sweep of `units` (set, candidate) pairs lays its windows' requests out by class and length first
// (sweep_ordered_kernels.hpp).  That saves the look at most requests of a window, and costs a launch and, per
// window and instance, bounds over its batches: it pays with windows of some hundred requests and candidates enough
// to hide a wavefront's trips to memory.  Measured, the other kernels' time over it, least and most of 4 to 256 slots, jittered
// fresh instances with three classes and loaded ones with eight, largest slack | shortest queue:
//   9000 candidates: windows of 128: 0.76-1.21 | 1.19, 256: 1.08-1.45 | 1.50-1.56, 512: 1.55-1.84 | 1.82-1.90, 4096: 4.68-6.96 | 3.87-4.03;
//   2000: 256: 0.91-1.12 | 1.28, 320: 1.23-1.61 | 1.70-1.99, 512: 1.06-1.55, 1024: 1.37-2.26, 16,384: 2.56-3.76 | 2.39-3.17;
//   720: 256: 0.78-1.14 | 1.08-1.33, 320: 1.12-1.56, 512: 0.98-1.35, 1024: 1.05-1.38, 256 slots 0.90-1.04, 4096: 1.48-2.17 | 1.25-1.43;
//   500: 1024: 0.78-1.31, 2048: 1.11-1.60 | 1.25-1.46; 100: 2048: 0.97-1.50, 4096: 1.18-1.56 | 0.86-1.13, 16,384: 1.08-1.59; 1: 4096: 0.84-1.72.
// Where several sets are scored (Alg. 2, over growth chains of equal instances) few instances count: 720 candidates, three
// sets, windows of 256: 1.75.
constexpr bool sweep_lays_out(uint64_t units, uint32_t n_sets, uint32_t i_pad, uint64_t per_window, bool shortest_queue) {
  if (per_window < 256u || units < 64u) return false;
  if (units >= 1000u) return per_window > 256u || n_sets > 1u || units >= 4096u || shortest_queue;
  if (units >= 720u) return per_window > 256u && (i_pad <= 128u || per_window >= 2048u);
  if (units >= 400u) return per_window >= 2048u;
  return per_window >= 4096u && !shortest_queue;
}

// Whether the prefills of every batch are then summed up ahead, on every row of the tables (batch_ticks_kernel): a launch of some
// 0.8 us per 4096 requests and thousand rows, for which a settled batch costs a look-up.  Measured, without the sums over with
// them, fresh jittered instances and 516 rows / loaded ones and 1028: 64 slots, 1100 candidates: windows of 512: 0.99 / 1.00, 1024: 1.03 / 1.04,
// 4096: 1.21 / 1.19, 16,384: 1.72 / 1.49; 9000: 512: 1.05 / 1.05, 1024: 1.06 / 1.08, 4096: 1.21 / 1.22; 300: 4096: 1.28 / 1.20; 4 slots, 1100: 1024: 0.80,
// 4096: 1.00 / 0.85, 16,384: 1.41 / 1.06; 9000: 1.16 / 1.00, 16,384: 1.72 / 1.30.
constexpr bool sweep_sums_batches(uint32_t i_pad, uint64_t per_window) {
  return per_window >= (i_pad >= 32u ? 2048u : 16384u);
}

// The same for the distributor (assign_ordered_kernels.hpp, against the persistent kernel): the chain of windows
// is then one block's, which looks for the instances that count and bounds their slacks one after the other, so it pays
// with few slots, or with windows that are much to score.  Measured, the persistent kernel's time over it, some hundred windows,
// least and most of empty smooth and loaded jittered instances:
//   largest slack: 2 slots: windows of 11 to 16,384: 2.5-5.6; 8 slots: 32: 0.97-2.8, 48: 1.26-3.9, 512: 2.4-4.8, 16,384: 1.8-2.6; 16 slots: 256:
//   0.99-4.2, 512: 1.39-4.1, 16,384: 1.38-2.1; 64 slots: 1024: 0.82-2.8, 2048: 1.02-2.9, 4096: 1.36-3.3, 16,384: 1.04-1.4, 32,768: 0.43-0.53; 128
//   slots: 2048: 0.76-2.0, 4096: 1.14-2.5, 8192: 1.44-2.4, 16,384: 0.79-0.97; 256 slots: 4096: 0.97-1.55, 8192: 1.12-1.51.
//   Shortest queue: 8 slots: 11: 2.7, 512: 5.8; 64 slots: 11: 0.88, 16: 1.15, 64: 3.7, 4096: 5.6, 16,384: 2.1, 32,768: 0.73; 128 slots: 16: 1.00, 32: 1.57,
//   8192: 4.2, 16,384: 1.55; 256 slots: 11: 1.27, 128: 2.1, 4096: 3.4, 16,384: 2.1.
constexpr bool assign_lays_out(uint32_t i_pad, uint64_t per_window, bool shortest_queue) {
  if (shortest_queue) return per_window >= (i_pad <= 16u ? 11u : i_pad <= 64u ? 16u : 32u) && per_window <= 16384u;
  if (i_pad <= 2u) return per_window >= 11u && per_window <= 16384u;
  if (i_pad <= 8u) return per_window >= 48u && per_window <= 16384u;
  if (i_pad <= 16u) return per_window >= 512u && per_window <= 16384u;
  if (i_pad <= 64u) return per_window >= 2048u && per_window <= 16384u;
  return per_window >= (i_pad <= 128u ? 4096u : 8192u) && per_window <= 8192u;
}

}  // namespace maaso
