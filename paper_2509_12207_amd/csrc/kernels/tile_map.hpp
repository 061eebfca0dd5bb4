// Which output tile a workgroup of a product computes.
#pragma once

#include <hip/hip_runtime.h>

namespace ug {
namespace {

constexpr int kXcds = 8;
constexpr int kGroupM = 8;
// s_waitcnt lgkmcnt(0) with the vmcnt and expcnt fields at their maxima
constexpr int kWaitLdsOnly = 15 | (3 << 14) | (7 << 4) | (0 << 8);

// Workgroups are dispatched round-robin over the XCDs: each takes a contiguous
// band of tiles, walked in groups of kGroupM tile rows.
__device__ __forceinline__ void tile_of(int wg, int tiles_m, int tiles_n, int* tm, int* tn) {
  const int total = tiles_m * tiles_n;
  const int x = wg % kXcds;   // XCDs below total % kXcds have one tile more
  const int id = x * (total / kXcds) + min(x, total % kXcds) + wg / kXcds;
  const int group = kGroupM * tiles_n;
  const int first_m = (id / group) * kGroupM;
  const int gm = min(tiles_m - first_m, kGroupM);
  const int r = id % group;
  *tm = first_m + r % gm;
  *tn = r / gm;
}

}  // namespace
}  // namespace ug
