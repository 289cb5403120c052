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

}  // namespace maaso
