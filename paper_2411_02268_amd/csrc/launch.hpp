// How many workgroups one launch may have (host; no HIP in here).
#pragma once
#include <algorithm>
#include <cstdint>

namespace mgcd {

// HIP takes fewer threads than this per grid dimension.
constexpr int64_t GRID_THREADS = (int64_t)1 << 32;

// Calls launch(first, count) for consecutive slices of `blocks` workgroups of `threads`
// threads, each small enough for one launch.  Kernels with several threads per row, chunk
// or community go through it: there are up to 2^31 of each.
template <typename F>
inline void launch_slices(int64_t blocks, int threads, F &&launch, int64_t limit = GRID_THREADS) {
  const int64_t most = (limit - 1) / threads;
  for (int64_t first = 0; first < blocks; first += most)
    launch(first, (unsigned)std::min<int64_t>(most, blocks - first));
}

}  // namespace mgcd
