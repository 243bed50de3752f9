// Tiles of the reducing line launches (host code, no HIP).
#pragma once

#include <algorithm>
#include <cstdint>

namespace helm {

// Tiles of `extent` lines that `groups` groups of blocks take along a reduced
// index, `step` lines per iteration of a block and at least `tmin` lines per tile:
// the fewest iterations in rounds of R resident blocks, a block's start and its
// partial sums counted as 0.7 of an iteration, among at most `most` blocks (or one
// tile per group).  A larger number of tiles has to be 2% better.
// Candidates are the distinct tile lengths, about 2 sqrt(extent) of the `extent`
// numbers of tiles: the search runs on the host in every eager solve, and over all
// numbers it took 33 us at 2049 modes and one right-hand side (now 1.6 us; a replay
// of a captured solve does not search).
// visited, if given, receives the number of candidates.
template <class I>
inline void reduce_tiles_as(I extent, I groups, I step, I tmin, I R, I most, int* tile, int* ntiles, int* visited) {
  double best = 1e300;
  int seen = 0;
  for (I n = 1; n <= extent && (n == 1 || groups * n <= most);) {
    I t = std::max((extent + n - 1) / n, tmin);
    t = (t + step - 1) / step * step;
    const I nt = (extent + t - 1) / t;
    const double cost = (double)((groups * nt + R - 1) / R) * ((double)(t / step) + 0.7);
    ++seen;
    if (cost < 0.98 * best) {
      best = cost;
      *tile = (int)t;
      *ntiles = (int)nt;
    }
    if (t < tmin + step) break;                // the shortest tiles
    n = (extent + t - step - 1) / (t - step);  // the next shorter ones
  }
  if (visited) *visited = seen;
}

inline void reduce_tiles(int64_t extent, int64_t groups, int64_t step, int64_t tmin, int64_t R, int64_t most,
                         int* tile, int* ntiles, int* visited = nullptr) {
  // (32-bit divisions where nothing can exceed them)
  if (groups < (1 << 30) && groups * (extent + step) + R < (int64_t(1) << 31))
    reduce_tiles_as<uint32_t>((uint32_t)extent, (uint32_t)groups, (uint32_t)step, (uint32_t)tmin, (uint32_t)R,
                              (uint32_t)most, tile, ntiles, visited);
  else
    reduce_tiles_as<int64_t>(extent, groups, step, tmin, R, most, tile, ntiles, visited);
}

}  // namespace helm
