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

}  // namespace maaso
