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

}  // namespace maaso
