"""Rays per tile of a scene's hidden-32 objects (scene_tile, scene_tile_low in
paper_2302_01838_amd/csrc/vmap_internal.h), evaluated on the host: the tiles of any number of pairs fit
the workspace's list, the shortest tile that does is the start, and the tile grows with the pairs."""
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
              const int max_pairs = max_rays / share;
              const int low = scene_tile_low(round, max_pairs, max_tiles - n);
              const int longest = low > kSceneRounds * round ? low : kSceneRounds * round;
              for (int part : {1, 2, 7, 1000}) {
                const int pairs = max_pairs / part, tile = scene_tile(low, longest, pairs);
                std::printf("%d %d %d %d %d %d %d %d %d %d\n", round, rpt, wide, max_pairs, n, max_tiles, low, longest, pairs, tile);
              }
            }
          }
  return 0;
}
"""


def test_scene_tiles_fit_and_follow_the_pairs(tmp_path):
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
    for rnd, rpt, wide, max_pairs, n, max_tiles, low, longest, pairs, tile in rows:
        what = (rnd, rpt, wide, max_pairs, n, pairs, low, tile)
        bound = lambda t: -(-pairs // (min(t, wide) if wide else t)) + n
        assert bound(tile) <= max_tiles, what
        assert low % rnd == 0 and low < max(rpt, wide) + rnd, what
        assert low <= tile <= longest and tile % low == 0, what
        if low > rnd:  # a shorter one would not fit
            assert -(-max_pairs // (low - rnd)) + n > max_tiles, what
        # as many tiles as forward mode holds workgroups, or the shortest tile
        assert tile == low or pairs // tile >= 1024, what
        assert 2 * tile > longest or pairs // (2 * tile) < 1024, what
