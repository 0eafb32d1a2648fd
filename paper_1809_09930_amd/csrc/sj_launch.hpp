// Launch sizes.  A dispatch holds fewer than 2^32 work-items: a launch of one
// thread per element covers every point set (n < 2^32), one of several threads
// per cell, list or work unit does not, and either strides or is cut here.
// Plain C++ (constexpr functions are device functions too).
#pragma once

#include <algorithm>
#include <cstdint>

namespace sj {

constexpr uint32_t kLaunchBlock = 256;          // threads of the strided kernels' workgroups
constexpr uint64_t kLaunchThreads = 1ull << 31;  // most threads of one cut launch

// Workgroups of a grid-stride launch over `threads` threads' work: all of it at
// once up to 2^20 workgroups.
constexpr uint32_t stride_blocks(uint64_t threads) {
  return (uint32_t)std::min<uint64_t>((threads + kLaunchBlock - 1) / kLaunchBlock, 1u << 20);
}

// f(first unit, units) for launches of at most kLaunchThreads threads that cover
// n units of `threads` (a power of two) threads each.
template <class F>
void for_unit_launches(uint64_t n, uint32_t threads, F &&f) {
  const uint64_t most = kLaunchThreads / threads;
  for (uint64_t u = 0; u < n; u += most) f(u, std::min(most, n - u));
}

// Steps of `lanes` lanes over the entries [b0, b1) of a list, and a lane's entry at a
// step: false past the list.  (Totals of lists may come up to 2^32 - 1 entries, and
// lanes that share a wave step on to its longest list: positions in 32 bits would
// wrap to other lists' entries.)
constexpr uint32_t list_steps(uint32_t b0, uint32_t b1, uint32_t lanes) {
  return (uint32_t)(((uint64_t)(b1 - b0) + lanes - 1) / lanes);
}
constexpr bool list_entry(uint32_t b0, uint32_t b1, uint32_t step, uint32_t lanes, uint32_t lane,
                          uint32_t *i) {
  const uint64_t at = (uint64_t)b0 + (uint64_t)step * lanes + lane;
  *i = (uint32_t)at;
  return at < b1;
}

}  // namespace sj
