// Launch shapes of the attention kernels: host arithmetic without HIP.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace thin {

// A launch's threads per grid dimension are counted in 32 bits (2^24 workgroups
// of 256 are refused), so a longer row of workgroups takes several rows of a
// further dimension: x * rows >= blocks, x a multiple of `multiple`.
struct GridRows {
  int64_t x, rows;
};
inline GridRows grid_rows(int64_t blocks, int64_t threads, int64_t multiple = 1) {
  const int64_t most = (((int64_t)1 << 32) - 1) / threads / multiple * multiple;
  const int64_t rows = (blocks + most - 1) / most;
  const int64_t x = (blocks + rows - 1) / rows;
  return {(x + multiple - 1) / multiple * multiple, rows};
}

}  // namespace thin
