"""The tile grid of a launch over one domain, on the CPU: the kernel's quotient
t / ntx (the high half of t div) is exact for every tile, and grids for which
it would not be take the table."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <initializer_list>
#include "nplbm_internal.h"
using namespace nplbm;
int main() {
  // the widest and the tallest lattices that tiles are chosen for, powers of
  // two and their neighbours, one column, and grids beyond the bound
  const int n[][2] = {{4, 4}, {32, 4000}, {33, 9}, {64, 17}, {96, 100}, {4095, 700}, {4096, 700},
                      {4097, 700}, {838860, 4}, {419430, 8}, {36, 93000}, {60000, 55},
                      {2000000, 2000}, {8400000, 64}};
  for (auto &s : n)
    for (int ty : {4, 8, 12}) {
      TileArgs a{};
      tile_grid(s[0], s[1], ty, a);
      const uint64_t ntx = ((uint64_t)s[0] + 31) / 32, nty = ((uint64_t)s[1] + ty - 1) / ty;
      long wrong = 0;
      if (a.ntx) {
        wrong += a.ntx != ntx || a.ntile != ntx * nty || (uint64_t)a.per * 8 < a.ntile;
        for (uint64_t t = 0; t < a.ntile; ++t) wrong += (t * a.div >> 32) != t / ntx;
      }
      std::printf("%d %d %d %d %ld\n", s[0], s[1], ty, (int)a.ntx, wrong);
    }
}
"""


def test_quotients_are_exact(tmp_path):
    src, exe = tmp_path / "g.cpp", tmp_path / "g"
    src.write_text(SRC)
    subprocess.run(["g++", "-std=c++17", "-O2",
                    "-I", os.path.join(ROOT, "tests", "host_double"),
                    "-I", os.path.join(ROOT, "paper_1904_12553_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    rows = [[int(v) for v in line.split()] for line in subprocess.run(
        [str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()]
    assert len(rows) == 42 and all(r[4] == 0 for r in rows), rows
    table = {(r[0], r[1]) for r in rows if r[3] == 0}
    assert table == {(4, 4), (32, 4000), (2000000, 2000), (8400000, 64)}
