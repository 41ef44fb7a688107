"""CPU test of the workgroup -> tile mappings (csrc/tile_map.h), compiled with the host compiler: over numbers of (batch, head) pairs and tiles
every tile has exactly one workgroup, no XCD has more tiles than another but for the granularity they are dealt out in, pairs
that need not be shared stay on one XCD, and an interleaved order never goes back to a longer rank.  The division that the mappings
use is compared with the compiler's."""

import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2407_17678_amd", "csrc")

DRIVER = r"""
#include <algorithm>
#include <cstdio>
#include <set>
#include <utility>
#include "tile_map.h"
using namespace s2;
static int check(bool ok, const char* what, int P, int T, int G, int w) {
  if (!ok) std::printf("%s: %d pairs, %d tiles, group %d, workgroup %d\n", what, P, T, G, w);
  return ok ? 0 : 1;
}
int main() {
  // every quotient changes at a multiple of d: there, on either side of it, and at the ends of the range
  for (long d = 1; d < (1l << 31); d += 1 + d / 37)
    for (long q = 0; q * d < (1l << 31); q += 1 + q / 5)
      for (long n : {q * d - 1, q * d, q * d + d - 1, (1l << 31) - 1 - q})
        if (n >= 0 && n < (1l << 31) && (int)n / fast_div((uint32_t)d) != (int)(n / d)) {
          std::printf("%ld / %ld\n", n, d);
          return 1;
        }
  for (int P = 1; P <= 77; ++P)
    for (int T : {1, 2, 3, 5, 8, 13, 31, 32, 33, 62, 63, 64, 65, 66, 127, 128, 129, 130, 131, 257})
      for (int G : {0, 1, 4, 5, 6}) {  // 0: interleaved; 4, 5: whole sequences, where an XCD has few and very many slots; 6: rows against a cache
        std::set<std::pair<int, int>> seen;
        int count[8] = {}, last[8] = {};
        const RowMap rows = row_map(P, T, G > 4 ? 4 : G, G == 6 ? kRowsOfCache : P & 1 ? kDenseRows : kSparseRows, G == 5 ? 1 << 20 : 64);
        const KeyMap keys = key_map(P, T);
        const int grid = (int)(G ? rows.grid() : keys.grid());
        if (check(grid % 8 == 0, "grid", P, T, G, grid)) return 1;
        for (int w = 0; w < grid; ++w) {
          int bh = -1, rank = -1;
          if (!(G ? map_workgroup(rows, w, bh, rank) : map_workgroup_interleaved(keys, w, bh, rank))) continue;
          const int x = w & 7;
          if (check(bh >= 0 && bh < P && rank >= 0 && rank < T, "range", P, T, G, w)) return 1;
          if (check(seen.insert({bh, rank}).second, "twice", P, T, G, w)) return 1;
          if (check(bh >= P / 8 * 8 || bh % 8 == x, "XCD", P, T, G, w)) return 1;
          // (the longest tiles of all pairs first, of the left-over ones too)
          if ((!G || (G == 5 && (P % 8 > 4 || (P % 8 && P > 39)))) && check(rank >= last[x], "order", P, T, G, w)) return 1;
          last[x] = rank;
          ++count[x];
        }
        if (check((int)seen.size() == P * T, "missing", P, T, G, grid)) return 1;
        // at most a run more, and the last run may be short
        const int most = *std::max_element(count, count + 8), least = *std::min_element(count, count + 8);
        if (check(most - least <= (P % 8 ? 1 << deal_run_shift(T) : 0), "balance", P, T, G, grid)) return 1;
      }
  // as many workgroups as 32 bits hold, and a few more: grids are counted in 64, and never less than the tiles
  for (int T : {64, 65, 129, 131, 8193})
    for (int left = 0; left < 8; ++left) {
      const int P = (int)((1ll << 31) / T / 8 * 8) + left;
      const long long rows = row_map(P, T, 1, kSparseRows, 64).grid(), keys = key_map(P, T).grid(), tiles = 1ll * P * T;
      if (check(rows >= tiles && rows <= tiles + 64 && keys >= tiles && keys <= tiles + 4ll * P + 64, "far", P, T, 0, 0)) return 1;
    }
  std::printf("mapped\n");
  return 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_every_tile_has_one_workgroup(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", CSRC, str(src), "-o", str(exe)], check=True, capture_output=True, text=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout == "mapped\n", r.stdout
