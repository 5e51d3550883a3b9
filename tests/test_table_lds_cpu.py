"""LDS of the training step's tile table (table_layout in paper_2302_01838_amd/csrc/vmap_internal.h),
evaluated on the host: what the tile kernel writes lies inside what its launch asks for, for every
wave count a launch accepts and batch sizes on both sides of each form of the table. Up to 64
objects a wave writes all three arrays (first tiles, ray offsets, object ids); beyond that the last
two only if the layout keeps them."""
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
  for (int bf = 0; bf <= 1; ++bf)
    for (int nw = 1; nw <= (bf ? 8 : 4); ++nw)
      for (int n : {1, 3, 4, 50, 63, 64, 65, 400, 600, kTableMaxObjects}) {
        const int base = lds_layout(32, bf != 0, nw).total;
        const TableLayout T = table_layout(base, n);
        std::printf("%d %d %d %d %d %d %d\n", bf, nw, n, base, T.pitch, T.rays ? 1 : 0, T.total);
      }
  return 0;
}
"""


def test_table_writes_lie_inside_the_launch(tmp_path):
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
    assert len(rows) == 12 * 10
    for bf, nw, n, base, pitch, rays, total in rows:
        what = (bf, nw, n)
        assert base % 16 == 0 and pitch % 4 == 0 and pitch >= n + 1, what
        end = base + 4 * (n + 1)                              # first tiles
        if n <= 64 or rays:
            end = max(end, base + 4 * (pitch + n + 1), base + 4 * (2 * pitch + n))  # offsets, ids
        assert end <= total, what
        assert total + 32 <= 160 * 1024, what                 # and the scan's eight static words
        if n <= 64:
            assert rays, what                                 # a workgroup's later tiles read them
