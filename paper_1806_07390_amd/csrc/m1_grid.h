// m1_grid.h -- host rules for grids of blocks (no device code).
#pragma once

#include <stdint.h>

#include <algorithm>

namespace fm1 {

// Blocks of a kernel that strides over the zones and writes one diagnostics partial per block:
// `need` blocks hold every zone once; at most as many as the step kernel's tiling has
// (`step_blocks`), but never fewer than per_cu on each of the device's compute units (the step
// kernel's few long blocks would leave the chip idle), and no more than the scratch has entries.
inline int64_t stride_blocks(int64_t need, int64_t step_blocks, int64_t entries, int per_cu, int cus) {
  const int64_t least = (int64_t)per_cu * (cus > 0 ? cus : 256);
  return std::max<int64_t>(1, std::min(std::min(need, entries), std::max(step_blocks, least)));
}

}  // namespace fm1
