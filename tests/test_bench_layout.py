"""bench.py picks the rows of its tables by the layout the library chooses: the rule it mirrors is the library's own."""
import subprocess

import bench
from paper_2505_23949_amd import build as hip_build

PROGRAM = r"""
#include "launch.hpp"
#include <cstdio>
using namespace tsenor_dev;
int main() {
  for (int M : {4, 8, 16, 32, 64})
    for (int fp32 : {0, 1})
      for (int iters : {1, 150, 151, 300})
        for (long n : {1L, 256L, 257L, 1024L, 1799L, 1800L, 2048L, 2049L, 3072L, 3073L, 8192L, 8193L, 12288L, 12289L, 49152L, 49153L,
                       62000L, 62001L, 65536L, 65537L, 102400L, 102401L, 114688L, 114689L, 1000000L}) {
          const bool team = n < team_below_blocks(M), small = team || (M <= 32 && small_tiles_win(M, fp32, false, iters, n));
          std::printf("%d %d %d %ld %s\n", M, fp32, iters, n,
                      !small ? "large" : team ? "team" : n < finest_tiles_below_blocks(M) ? "finest" : "small");
        }
}
"""


def test_layout_of_is_the_librarys_rule(tmp_path):
    source, program = tmp_path / "rule.hip", tmp_path / "rule"
    source.write_text(PROGRAM)
    subprocess.run([hip_build.HIPCC, *hip_build.FLAGS, f"-I{hip_build.CSRC}", "-o", str(program), str(source)], check=True,
                   stderr=subprocess.DEVNULL)
    lines = subprocess.run([str(program)], check=True, capture_output=True, text=True).stdout.split("\n")
    cases = [line.split() for line in lines if line]
    assert len(cases) == 5 * 2 * 4 * 25
    for M, fp32, iters, n, layout in cases:
        assert bench.layout_of(int(M), fp32 == "1", int(n), int(iters)) == layout, (M, fp32, iters, n)
