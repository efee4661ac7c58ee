"""Row splits of the rank <= 16 right product, from the plan compiled with the
host compiler: at padded rank 4 a small grid keeps splits of 32 rows (few long
ones make the whole call wait), a grid of many column tiles or a higher rank
does not get more splits for it, and the blocks of one matrix never exceed one
round.
"""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#define __host__
#define __device__
#include "plan.hpp"
#include <cstdio>
int main() {
  for (int rp : {4, 8, 16})
    for (long m : {128, 256, 512, 1024, 4096, 65536})
      for (long n : {64, 128, 256, 512, 1024, 4096, 12288}) {
        const occ::Tiling t = occ::make_tiling(m, n, rp);
        std::printf("%d %ld %ld %d %d\n", rp, m, n, t.sq, t.q_rows);
      }
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_splits_of_small_and_wide_grids(tmp_path):
    src, exe = tmp_path / "splits.cpp", tmp_path / "splits"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2301_09830_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    seen = {}
    for line in subprocess.run([str(exe)], capture_output=True, text=True, check=True).stdout.split("\n")[:-1]:
        rp, m, n, sq, q_rows = map(int, line.split())
        seen[rp, m, n] = sq
        assert sq * q_rows >= m and -(-n // 128) * sq <= 511
    for rp, few in ((4, (4, 8, 16)), (8, (2, 4, 8)), (16, (2, 4, 8))):
        assert (seen[rp, 128, 128], seen[rp, 256, 256], seen[rp, 512, 512]) == few
        assert seen[rp, 256, 4096] == 4 and seen[rp, 1024, 1024] == 16 and seen[rp, 4096, 1024] == 32
