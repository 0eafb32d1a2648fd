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

}  // namespace sj
