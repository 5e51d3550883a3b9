"""Where the tile kernel's end-of-tile gradient copies lie (paper_2302_01838_amd/csrc/vmap_internal.h),
evaluated on the host: in the staging space, and of four waves' four copies the last over the weights,
which the next tile fetches again. That one must end before the encoding matrix, loaded once per
workgroup."""
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
    for (int nw = 1; nw <= 8; ++nw) {
      const LdsLayout L = lds_layout(32, bf != 0, nw);
      std::printf("%d %d %d %d %d %d %d\n", bf, nw, scratch_copies(nw), kRedCopyBytes, L.B_off, L.scratch_off, L.total);
    }
  std::printf("%d\n", n_params_of(32));
  return 0;
}
"""


def test_gradient_copies(tmp_path):
    if not os.path.exists(HIPCC) or shutil.which("g++") is None:
        pytest.skip("hipcc not available")
    src = tmp_path / "drv.cpp"
    src.write_text(DRIVER)
    exe = tmp_path / "drv"
    subprocess.run([HIPCC, "-std=c++17", "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2302_01838_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout.splitlines()
    params = int(out[-1])
    rows = [list(map(int, ln.split())) for ln in out[:-1]]
    assert len(rows) == 16
    for bf, nw, copies, copy_bytes, b_off, scratch_off, total in rows:
        assert copy_bytes >= 4 * params and copy_bytes % 16 == 0
        assert scratch_off + copies * copy_bytes <= total, (bf, nw)
        assert copies == {4: 3, 8: 4, 1: 1}.get(nw, 2)
        if nw == 4:
            assert copy_bytes <= b_off
