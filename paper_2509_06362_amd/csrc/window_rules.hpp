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

// Whether the windowed sweep of `units` (set, candidate) pairs lays its windows' requests out by class and length first (sweep_ordered_kernels.hpp).
// That saves the look at most requests of a window, and costs a launch of some 10 us, with the batches' sums another, and per window and instance
// bounds over its batches.  It pays with windows of some hundred requests, with candidates enough to hide a wavefront's trips to memory, and with
// windows enough to earn the launches and the first windows, in which most instances still admit: some 12 * 2^20 requests times candidates.
// Measured, the other kernels' time over it, least and most of empty, fresh, loaded and stressed instances, smooth and jittered profiles, three and
// eight classes, by number of windows, largest slack:
//   64 slots: 64 candidates, windows of 4096: 1: 0.60-1.05, 4: 0.81-1.23, 8: 1.06-1.53, 16: 1.25-1.85; 512, of 2048: 1: 0.68-0.93, 8: 0.99-1.44, 16:
//   1.11-1.74; 512, of 4096: 2: 0.81-1.31, 4: 1.15-1.52; 1024, of 320: 4: 1.00-1.30, 8: 1.15-1.43; of 512: 8: 0.95-1.30, 16: 1.01-1.39; of 1024: 8:
//   0.96-1.46, 16: 1.15-1.62; of 2048: 2: 0.76-1.44, 4: 0.99-1.72; of 4096: 1: 0.80-1.31, 2: 1.02-1.72; of 16,384: 1: 0.84-2.02, 2: 1.05-2.73; 4096,
//   of 256: 8: 0.92-1.01, 16: 0.97-1.07, 64: 1.13-1.28; of 512: 4: 0.92-1.33, 8: 1.05-1.43; of 1024: 2: 1.06-1.70; of 4096: 1: 1.43-3.10, 16:
//   4.25-6.73; 8192, of 512: 4: 1.08-1.52; of 4096: 1: 1.92-4.15.
//   4 slots: 4096, of 512: 8: 0.99-1.10, 16: 1.20-1.37.  256 slots: 64, of 16,384: 4: 0.89-1.98; 1024, of 512: 4: 1.00-1.53; of 2048: 2: 1.04-1.78.
//   Shortest queue, 64 slots: 512, of 2048: 1: 1.04-1.08; 1024, of 320: 1.09-1.13, of 4096: 1.38-1.60; 4096, of 512: 1.05-1.22.
// Several sets (Alg. 2: growth chains of equal instances against three): 1134 deployments and sets, windows of 256: 16: 1.03, 32: 1.14; of 512: 16:
// 1.00, 32: 1.12; 2160, of 256: 16: 1.00, 64: 1.28; of 4096: 1: 1.00; 558 and fewer, of 4096: 16: 0.79-1.08, 32: 0.92-1.6; 1080 to 4320, of 257
// to 400: 4: 0.89-1.05, 7: 0.99-1.10, 11: 1.09-1.17, 15: 1.17-1.24; 954 to 1890, of 478 to 937: 9 to 15: 0.97-1.21, 6 to 8: 0.97-1.07; 882, of 478: 10: 1.13; 738: 0.95-1.02.
// 116 calls drawn from the timed ranges, two inputs each, largest slack, by candidates and number of windows: below 400: 1 and 2: 0.36-1.23, mean 0.66,
// 4 to 10, 12 slots and more: 0.99-3.8, fewer: 0.77-1.14; 400 to 999: 1: 0.52-1.33, mean 0.78, 2: 0.65-1.24, 3 to 6: 0.78-1.65; 1000 to 1999: 1 and 2: 0.58-1.21,
// mean 0.93, 80 slots and more 0.75-1.92, mean 1.3; 3 to 8: 1.09-2.03, four slots 0.90; 2000 to 3999, 1 and 2, windows below 1024: 0.57-1.13, above: 0.87-1.54; 4 to 7: 1.1-1.8; more, 1: 1.01-1.95,
// three slots 0.87.  The line was laid where the mean of a shape over these is above one and its least, as a rule, not below 0.8.
constexpr bool sweep_lays_out(uint64_t units, uint32_t n_sets, uint32_t i_pad, uint64_t per_window, uint64_t n_windows, bool shortest_queue) {
  if (per_window < 256u || units < 64u) return false;
  const bool candidates = units >= 1000u  ? per_window > 256u || n_sets > 1u || units >= 4096u || shortest_queue
                          : units >= 720u ? per_window > 256u && (i_pad <= 128u || per_window >= 2048u)
                          : units >= 400u ? per_window >= 2048u
                                          : per_window >= 4096u && !shortest_queue;
  if (!candidates) return false;
  if (n_sets > 1u && units < 2000u && per_window >= 1024u) return n_windows >= 32u && units >= 400u;
  if (n_sets > 1u && per_window > 256u && (per_window < 465u ? n_windows >= 7u : per_window < 1024u && n_windows >= 9u && units >= 850u)) return true;
  if (n_windows >= (units < 400u ? 32u : 16u)) return true;
  if (n_sets == 1u && per_window > 256u) {  // (the drawn calls above)
    if (n_windows >= (units < 400u    ? i_pad >= 12u ? 4u : 32u
                      : units < 2000u ? i_pad >= 16u ? 3u : units < 1000u ? 5u : 6u
                      : units < 4000u ? i_pad >= 8u ? 4u : 6u
                                      : i_pad >= 8u ? 1u : 3u))
      return true;
    if (units >= 1000u && (i_pad >= 80u || (units >= 2000u && per_window >= 1024u && i_pad >= 5u))) return true;
  }
  uint64_t gain = 1;
  if (shortest_queue) gain = i_pad >= 64u ? 8u : i_pad >= 16u ? 4u : per_window >= 1024u ? 2u : 1u;
  else if (per_window > 256u && i_pad > 8u) gain = i_pad > 128u ? 4u : per_window >= 1024u ? 2u : 1u;
  const uint64_t chains = units * n_windows * gain;
  if (per_window >= 16384u) return n_windows >= 4u || chains * (per_window < 32768u ? per_window : 32768u) >= 45u << 20;
  // (500 candidates x 16 slots, one window of 16,000: 0.68)
  return chains * (per_window < 4096u ? per_window : 4096u) >= (per_window > 256u && per_window < 465u ? 6u << 20 : 12u << 20);
}

// Whether the prefills of every batch are then summed up ahead, on every row of the tables (batch_ticks_kernel): a launch of some 0.8 us per 4096
// requests and thousand rows and what it waits for, for which a settled batch costs a look-up, whatever the number of candidates.  Measured, without
// the sums over with them, 64 to 4096 candidates, by number of windows: 64 slots, windows of 2048: 1: 0.68-0.85, 4: 0.87-0.99, 8: 0.98-1.17, 16:
// 1.05-1.42, 64: 1.09-1.78; 4096: 2: 0.87-0.97, 4: 0.97-1.24, 16: 1.11-1.83; 16,384: 1: 0.95-1.30, 4: 1.15-2.15; 256 slots: 2048: 8: 0.97-1.08, 64:
// 1.04-1.36; 16,384: 1: 0.95-1.21; 4 slots: 2048: 64: 0.69-0.95; 4096: 16: 0.83-1.19; 16,384: 1: 0.94-1.31, 4: 1.12-2.29.
constexpr bool sweep_sums_batches(uint32_t i_pad, uint64_t per_window, uint64_t n_windows) {
  return per_window >= (i_pad >= 32u ? 2048u : 16384u) && per_window * n_windows >= 16384u;
}

// The same for the distributor (assign_ordered_kernels.hpp, against the persistent kernel): the chain of windows is then one block's, which looks for
// the instances that count and bounds their slacks one after the other.  It pays with few slots, or where a placement is overloaded and most windows
// admit nothing, which takes a stream long enough: with many different instances below or at their capacity it is slower.  A call of a few windows is
// mostly the launches: 26 us, the persistent kernel's 34.  Measured, the persistent kernel's time over it, least and mean of empty and loaded
// instances, smooth and jittered profiles, arrivals from a tenth of what the placement serves to many times that, by number of windows:
//   largest slack: 2 slots: windows of 11: 1: 1.18 1.31, 1024: 1.46 3.36; 16,384: 1: 1.05 1.13, 256: 3.67 3.73; 4 slots: 64: 1024: 1.00 3.03; 4096:
//   1: 1.23 1.29; 16,384: 2: 0.93 0.98, 32: 1.62 1.77; 8 slots: 64: 256: 0.68 1.57; 256: 128: 0.89 1.45; 512: 64: 0.93 1.71, 1024: 1.07 3.20; 4096:
//   1: 1.15 1.21, 128: 1.05 1.75; 8192: 64: 0.80 1.81, 128: 1.47 1.99; 16 slots: 1024: 128: 0.88 1.34; 2048: 16: 0.98 1.15, 64: 0.97 1.46; 4096: 8:
//   0.85 1.04, 32: 1.06 1.24; 8192: 128: 0.79 1.33, 256: 1.43 2.88; 32 slots: 2048: 4: 0.99 1.25, 16: 0.72 1.12, 64: 0.99 1.31; 8192: 256: 1.02 2.61;
//   64 slots: 2048: 2: 1.04 1.14, 64: 0.64 0.97, 256: 0.95 1.54, 1024: 1.05 2.66; 4096: 1: 0.89 1.02, 64: 0.75 1.17, 128: 1.19 1.44, 1024: 1.38 3.32;
//   16,384: 256: 0.85 1.95; 128 slots: 4096: 128: 0.79 1.15, 256: 1.30 1.59; 16,384: 256: 0.96 1.52; 256 slots: 8192: 256: 0.83 1.23, 512: 1.32 1.58.
//   Shortest queue: 2 slots: 11: 1: 1.17 1.30; 8 slots: 11: 64: 0.86 1.15; 32: 1.04 1.99; 16,384: 32: 0.66 1.19, 64: 1.24 1.86; 16 slots: 32: 64:
//   0.78 1.15; 128: 1.10 1.50; 16,384: 128: 1.42 1.91; 32 slots: 64: 0.89 1.69; 256: 1.16 1.72; 16,384: 128: 0.95 1.62, 256: 1.75 3.39; 64 slots: 64:
//   0.77 1.27; 256: 1024: 0.92 2.84; 1024: 1.15 1.40; 4096: 1: 0.92 1.04, 4: 1.02 1.19; 16,384: 2: 0.88 0.94, 8: 1.00 1.06; 128 slots: 64: 8: 0.85
//   1.13, 256: 0.73 1.62; 256: 8: 0.91 1.27; 512: 4: 1.00 1.35; 4096: 4: 0.94 1.14, 8: 1.16 1.29; 256 slots: 512: 8: 0.91 1.21, 16: 0.99 1.47; 1024:
//   8: 0.97 1.26; 8192: 8: 1.17 1.34.
// 80 calls drawn from the timed ranges, arrivals of 400 to 5000 a second, by number of windows: largest slack: 1 to 5: 1.01 to 1.39 (one 0.8), more: 1.00-2.9,
// but 9 to 16 slots, windows above 4096, 7 and 14: 0.8-1.0, 62: 1.7, and 43 slots of 10,639, 17: 0.85.  Shortest queue: windows of 17 to 43, up to 64 slots, 38 to 65: 0.69-0.88, 348:
// 0.78-1.19, 725: 0.6, 958: 3.0, 1000: 5.6, of 57: 2.3; 67 to 84 slots, of 33 to 41: 0.67-3.2, mean 1.2, of 46 and more: 1.04-5.8; 130 and more, of 39 and more: 1.1-1.9; windows of
// hundreds and thousands, up to 128 slots: 0.9-1.5 (one 0.77), 130 and more: 1: 0.67-1.6, 2: 0.8-1.38, 3: 1.2-2.2, mean 1.1 of 1 and 2.
// The line was laid where the mean of a shape is above one (below it remain 8 slots, windows of 48 to 255, at capacity: 0.64 to 0.9, and a few more).
constexpr bool assign_lays_out(uint32_t i_pad, uint64_t per_window, uint64_t n_windows, bool shortest_queue) {
  if (per_window < 11u || per_window > 16384u) return false;
  if (i_pad <= 2u) return true;
  if (shortest_queue) {
    if (per_window <= 64u) {
      if (i_pad <= 8u) return true;
      if (i_pad <= 16u) return n_windows >= (per_window < 16u ? 512u : 128u) || per_window >= 32u;
      if (i_pad <= 32u) return (per_window >= 16u && n_windows >= 256u) || per_window >= 32u;
      if (i_pad <= 64u) return (per_window >= 16u && n_windows >= 512u) || per_window >= 48u;
      return per_window >= 32u;
    }
    return true;
  }
  if (i_pad <= 8u) return per_window >= 48u && (per_window <= 8192u || i_pad <= 4u || n_windows >= 8u || n_windows <= 3u);
  if (i_pad <= 16u) return per_window >= 512u && (per_window <= 4096u || n_windows >= 48u || n_windows <= 5u);
  if (i_pad <= 32u) return per_window >= 2048u;
  if (i_pad <= 64u) return per_window >= 2048u && (per_window <= 8192u || n_windows >= 64u);
  return per_window >= (i_pad <= 128u ? 4096u : 8192u) && per_window <= 8192u && (i_pad <= 128u || n_windows >= 256u);
}

}  // namespace maaso
