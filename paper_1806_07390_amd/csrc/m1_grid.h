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

// Whether a double 3-D step of a group count that 4 does not divide runs faster on the 3-D plane
// kernel (blocks of TM planes, one block of 8 waves per CU) than on the tiled kernel.  Both walk
// their planes one after the other, with about three planes' worth of start-up, so the time goes
// as rounds of blocks times planes + 3; the tiled kernel holds 8 waves per CU, and on spherical
// grids its time grows from the second wave per SIMD on.  The margin (in percent) is what the plane
// kernel's planes take more: over 254 grids (8^3 to 256 x 64 x 64, 1 to 18 groups) in each of four
// sets of options it was the slower one (tiled -> plane kernel, us) up to a ratio of
//   Cartesian: 109 % minmod, MC (8^3 x 3 37 -> 40), 118 % M1 speeds (10^3 x 1 61 -> 66), 127 % PPM
//     (10 x 10 x 11 x 1 RK2 135 -> 139); faster above (12^3 x 3 50 -> 40, 90 x 70 x 60 x 10 316 -> 213);
//   spherical: 118 % minmod (128 x 48 x 10 x 3 62 -> 66); other limiters and M1 speeds, whose
//     instantiation spills registers, 224 % where its blocks fill the chip (180 x 64 x 96 x 3 MC 701 ->
//     739) and 136 % where they are few (40 x 10 x 12 x 9 MC 91 -> 107; 32 x 8 x 16 x 9 at 173 % 126 ->
//     106), 241 % with PPM.
inline int64_t plane_kernel_margin(bool spherical, bool minmod, bool ppm, bool m1_speeds, int64_t blocks, int64_t cu) {
  if (!spherical) return ppm ? 130 : (m1_speeds ? 120 : 112);
  if (minmod && !m1_speeds) return 120;
  return ppm ? 245 : 150 + 75 * std::min(5 * blocks, 4 * cu) / (4 * cu);
}

inline bool plane_kernel_pays(int64_t c3_blocks, int c3_TM, int64_t tiled_blocks, int tiled_threads, int tiled_TM,
                              int n2, bool spherical, bool minmod, bool ppm, bool m1_speeds, int cus) {
  const int64_t cu = cus > 0 ? cus : 256;
  auto rounds = [](int64_t n, int64_t slots) { return (n + slots - 1) / slots; };
  const int64_t cost = rounds(c3_blocks, cu) * (std::min(c3_TM, n2) + 3);
  const int64_t waves = tiled_threads / 64 > 0 ? tiled_threads / 64 : 1;
  const int64_t r = spherical ? rounds(tiled_blocks * waves, 4 * cu)
                              : rounds(tiled_blocks, cu * std::max<int64_t>(1, 8 / waves));
  const int64_t tiled = r * (std::min(tiled_TM, n2) + 3);
  return 100 * tiled >= plane_kernel_margin(spherical, minmod, ppm, m1_speeds, c3_blocks, cu) * cost;
}

}  // namespace fm1
