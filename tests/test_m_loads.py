"""Which elements of M one vector load may touch, checked on the host (the rule
the kernels use, compiled with the host compiler): never an element outside the
array, and in the row-sparse step never one outside the listed row, whose
neighbours in M belong to the caller.
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
  long passed = 0;
  for (int listed = 0; listed < 2; ++listed)
    for (int m = 1; m <= 4; ++m)
      for (int n = 1; n <= 40; ++n)
        for (int ldm = n; ldm <= n + 20; ++ldm)
          for (int row = 0; row < m; ++row)
            for (int c = 0; c < n; ++c)
              for (int w : {4, 8, 16}) {
                if (!occ::m_load_may_pass(listed != 0, row, m, ldm, n, c, w)) {
                  if (c + w <= n) return std::puts("a load inside the row is refused"), 1;
                  continue;
                }
                if (row * ldm + c + w > (m - 1) * ldm + n) return std::puts("past the array"), 1;
                if (listed && c + w > n) return std::puts("past a listed row"), 1;
                passed += c + w > n;
              }
  std::printf("%ld\n", passed);
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_loads_stay_inside_the_array_and_the_listed_rows(tmp_path):
    src, exe = tmp_path / "loads.cpp", tmp_path / "loads"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(ROOT, "paper_2301_09830_amd", "csrc"),
                    str(src), "-o", str(exe)], check=True)
    run = subprocess.run([str(exe)], capture_output=True, text=True)
    assert run.returncode == 0, run.stdout
    assert int(run.stdout) > 0      # rows that are not listed do take loads past their end

