"""The tile search of the reducing line launches (csrc/line_tiles.h, compiled
here on its own): the tiles of a search over every number of tiles, from a few
candidates, because it runs on the host in every eager solve."""

import os
import subprocess

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1809_03808_amd", "csrc")

DRIVER = r"""
#include <cmath>
#include <cstdio>
#include "line_tiles.h"

// every number of tiles
static void all(int64_t extent, int64_t groups, int64_t step, int64_t tmin, int64_t R, int64_t most, int* tile, int* nt) {
  double best = 1e300;
  for (int64_t n = 1; n <= extent && (n == 1 || groups * n <= most); ++n) {
    int64_t t = std::max((extent + n - 1) / n, tmin);
    t = (t + step - 1) / step * step;
    const int64_t k = (extent + t - 1) / t;
    const double cost = (double)((groups * k + R - 1) / R) * ((double)(t / step) + 0.7);
    if (cost < 0.98 * best) { best = cost; *tile = (int)t; *nt = (int)k; }
  }
}

int main() {
  long n = 0;
  for (int64_t extent : {3, 4, 5, 7, 8, 16, 61, 128, 129, 200, 257, 500, 513, 1023, 1024, 2049, 4096, 4097, 70000})
    for (int64_t groups : {1, 2, 3, 7, 16, 61, 129, 256, 500, 1024, 4096, 100000})
      for (int64_t step : {1, 2, 4, 8, 32, 256})
        for (int64_t least : {1, 4, 8})
          for (int64_t R : {256, 512})
            for (int64_t m : {1, 8}) {
              const int64_t tmin = std::min(least, extent);
              int t0 = -1, k0 = -1, t1 = -1, k1 = -1, seen = 0;
              all(extent, groups, step, tmin, R, m * R, &t0, &k0);
              helm::reduce_tiles(extent, groups, step, tmin, R, m * R, &t1, &k1, &seen);
              ++n;
              if (t0 != t1 || k0 != k1 || seen > 2 * std::sqrt((double)extent) + 2) {
                std::printf("extent %ld groups %ld step %ld tmin %ld R %ld m %ld: %d x %d, all %d x %d, %d seen\n",
                            (long)extent, (long)groups, (long)step, (long)tmin, (long)R, (long)m, t1, k1, t0, k0, seen);
                return 1;
              }
            }
  std::printf("%ld geometries\n", n);
  return 0;
}
"""


def test_tiles_of_the_whole_search_from_few_candidates(tmp_path):
    src, exe = tmp_path / "tiles.cpp", tmp_path / "tiles"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O2", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout
    assert int(out.stdout.split()[0]) == 19 * 12 * 6 * 3 * 2 * 2
