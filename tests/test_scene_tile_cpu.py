"""Rays per tile of forward launches without losses (forward_tile, scene_tile_low in
paper_2302_01838_amd/csrc/vmap_internal.h), evaluated on the host: the tiles of any number of rays fit the
work list, the shortest tile that does is the start, and of the tiles of up to eight rounds none has a
smaller estimate of its time."""
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
                const int rays = bound / part;
                for (int bf16 : {0, 1})
                  for (int waves : {2, 4})
                    std::printf("%d %d %d %d %d %d %d %d %d %d %d\n", round, rpt, wide, bound, n, max_tiles, low, rays,
                                bf16, waves, forward_tile(bf16 != 0, round, waves, low, rays, n));
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
    assert len(rows) == 5 * 7 * 3 * 5 * 3 * 3 * 4 * 4

    def cost(bf16, quads, most, k):
        if bf16:
            return (-(-quads // 256) * 256 + 3 * max(256, quads + 128)) * (4 * k + 1)
        return max(448, quads) * (2 * k + 1) if k <= 2 or k <= 6 and most <= 512 else None

    for rnd, rpt, wide, bound, n, max_tiles, low, rays, bf16, waves, tile in rows:
        what = (rnd, rpt, wide, bound, n, rays, low, bf16, waves, tile)
        assert -(-rays // (min(tile, wide) if wide else tile)) + n <= max_tiles, what
        assert low % rnd == 0 and low < max(rpt, wide) + rnd, what
        if low > rnd:  # a shorter one would not fit
            assert -(-bound // (low - rnd)) + n > max_tiles, what
        costs = {k: cost(bf16, (rays // (k * rnd) + (n + 1) // 2) * waves // 4, (rays // (k * rnd) + n) * waves // 4, k)
                 for k in range(low // rnd, 9)}
        costs = {k: c for k, c in costs.items() if c is not None}
        best = min(costs.values()) if costs else None
        assert tile == (rnd * max(k for k, c in costs.items() if c == best) if costs else low), what
        if rays // low + n <= 128:  # few tiles: no longer than they need be
            assert tile == low, what
