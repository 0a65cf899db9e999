"""Host check (not a GPU test) of the order in which the blocks of FP64 maps are
dealt out: in every row of the grid each job once, and for any number of jobs each of
the 32 positions of the round robin gets every job about equally often; the launch
has the jobs along x, so that no position is left with the same chunks."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SRC = r"""
#include <cstdio>
#include <vector>
#include "dd_gauss.h"
int main() {
  int worst = 0;
  for (unsigned n : {1u, 7u, 12u, 16u, 28u, 32u, 44u, 64u, 96u, 384u}) {  // jobs
    const unsigned rows = 32 * n;
    std::vector<int> seen(32 * n, 0);
    for (unsigned y = 0; y < rows; ++y) {
      std::vector<int> once(n, 0);
      for (unsigned x = 0; x < n; ++x) {
        const unsigned j = dd::gauss_job_of(x, y, n);
        if (j >= n || once[j]++) return 1;
        ++seen[((unsigned long long)y * n + x) % 32 * n + j];
      }
    }
    // 32 n rows: n blocks of a job per position on average
    for (int s : seen) worst = s * 100 / (int)n > worst ? s * 100 / (int)n : worst;
  }
  printf("%d\n", worst);
}
"""


def test_blocks_are_spread(tmp_path):
    gxx = shutil.which("g++")
    if not gxx or not os.path.isdir("/opt/rocm/include/hip"):
        pytest.skip("no g++ or HIP headers")
    src = tmp_path / "blocks.cpp"
    src.write_text(SRC)
    exe = tmp_path / "blocks"
    subprocess.run([gxx, "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I",
                    os.path.join(ROOT, "paper_2507_00294_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True)
    worst = int(subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout)
    assert worst <= 200, worst  # at most twice its share of any job
