"""The left product's fp32 sums above rank 16 do not get longer where the plan
gives a block more columns (one matrix alone, whole rounds of blocks): a longer
sum is a larger error against float64.  The plan is compiled with the host
compiler and checked over shapes, against the splits it starts from.
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
using namespace occ;
// K-steps of a block of the splits that the search starts from
static int64_t start_steps(int64_t m, int64_t n, int rp, const Slots& sl) {
  const int64_t target = whole_rounds(L_SPLIT_BLOCKS, sl.p), tiles = cdiv(m, lp_block_rows(rp, false));
  int64_t w = L_MIN_COLS, sp;
  while (sp = clamp64(cdiv(target, tiles), 1, cdiv(n, w)), w > L_MIN_NARROW && tiles * sp < sl.p) w /= 2;
  return cdiv(cdiv(n, sp), L_KC);
}
int main() {
  long merged = 0, whole = 0;
  for (int rp : {32, 64, 128})
    for (int64_t slots : {256, 512, 768}) {
      Slots sl{slots, 512, 1024};
      for (int64_t m = 32; m <= 70000; m = m * 9 / 8 + 1)
        for (int64_t n = 32; n <= 13000; n = n * 9 / 8 + 1) {
          const Tiling t = make_tiling(m, n, rp, 1.0, sl, false);
          const int64_t steps = t.p_cols / L_KC, first = start_steps(m, n, rp, sl);
          if ((int64_t)t.sp * t.p_cols < n) return std::puts("columns left out"), 1;
          if (steps <= first) { whole += t.p_sub >= steps; continue; }
          ++merged;
          if (t.p_sub < 1 || t.p_sub > first) {
            std::printf("%ld x %ld rank %d: sums of %ld K-steps, %ld before\n", (long)m, (long)n, rp,
                        (long)std::min<int64_t>(t.p_sub, steps), (long)first);
            return 1;
          }
        }
    }
  std::printf("%ld %ld\n", merged, whole);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_sums_are_no_longer_than_the_first_splits(tmp_path):
    src, exe = tmp_path / "sums.cpp", tmp_path / "sums"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-I",
                    os.path.join(ROOT, "paper_2301_09830_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
    merged, whole = map(int, run.stdout.split())
    assert merged > 0 and whole > 0    # both kinds of plan were seen
