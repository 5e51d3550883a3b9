"""Rays per tile of forward launches without losses (forward_tile, scene_tile_low in
paper_2302_01838_amd/csrc/vmap_internal.h), evaluated on the host: the tiles of any number of rays fit the
work list, the shortest tile that does is the start, and of the tiles of up to eight rounds none has a
smaller estimate of the rounds that the chip's workgroup slots get."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = "/opt/rocm/bin/hipcc"

DRIVER = r"""
#include <cstdio>
#include "vmap_internal.h"
using namespace vmapi;
int main() {
  for (int round : {4, 8, 12, 24, 512})
    for (int rpt : {1, 8, 12, 24, 36, 48, 65536})
      for (int wide : {0, 8, 64})
        for (int max_rays : {1, 1000, 20000, 307200, 1 << 26})
          for (int n : {1, 50, 2000}) {
            const int least = wide > 0 && wide < rpt ? wide : rpt;
            const int max_tiles = (max_rays + least - 1) / least + n;  // of a stack of n objects
            for (int share : {1, 3, 100}) {
              const int bound = max_rays / share;
              const int low = scene_tile_low(round, bound, max_tiles - n);
              for (int part : {1, 2, 7, 1000}) {
                const int rays = bound / part, slots = part % 2 ? 1024 : 512;
                const int tile = forward_tile(round, low, rays, n, slots);
                std::printf("%d %d %d %d %d %d %d %d %d %d\n", round, rpt, wide, bound, n, max_tiles, low, rays, slots, tile);
              }
            }
          }
  return 0;
}
"""


def test_forward_tiles_fit_and_follow_the_rays(tmp_path):
    if not os.path.exists(HIPCC) or shutil.which("g++") is None:
        pytest.skip("hipcc not available")
    src = tmp_path / "drv.cpp"
    src.write_text(DRIVER)
    exe = tmp_path / "drv"
    subprocess.run([HIPCC, "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2302_01838_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    rows = [list(map(int, ln.split())) for ln in
            subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()]
    assert len(rows) == 5 * 7 * 3 * 5 * 3 * 3 * 4
    for rnd, rpt, wide, bound, n, max_tiles, low, rays, slots, tile in rows:
        what = (rnd, rpt, wide, bound, n, rays, low, tile)
        assert -(-rays // (min(tile, wide) if wide else tile)) + n <= max_tiles, what
        assert low % rnd == 0 and low < max(rpt, wide) + rnd, what
        if low > rnd:  # a shorter one would not fit
            assert -(-bound // (low - rnd)) + n > max_tiles, what
        assert tile % rnd == 0 and low <= tile <= max(low, 8 * rnd), what
        cost = lambda k: -(-(rays // (k * rnd) + (n + 1) // 2) // slots) * (2 * k + 1)
        if tile <= 8 * rnd:
            ks = range(low // rnd, 9)
            assert cost(tile // rnd) == min(map(cost, ks)), what
            assert all(cost(k) > cost(tile // rnd) for k in ks if k * rnd > tile), what  # the longest of equals
        if rays > 0 and -(-rays // low) + n <= slots:  # one round of the chip: no longer than it need be
            assert tile == low or tile > 8 * rnd, what
