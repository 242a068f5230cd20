"""Positions of the pooling kernel on values at the largest maps, on the host: its
walk ends, and reads inside the map."""
import os
import subprocess

from paper_2007_06563_amd import build

SRC = r"""
#include <stdio.h>
#include "kernels.hpp"
int main() {
  const uint32_t ahead = 8;
  for (uint32_t hw : {1u, 2u, 15u, 16u, 17u, 0x7FFFFFEFu, 0x7FFFFFF0u, 0x7FFFFFF1u, 0x7FFFFFFEu, 0x7FFFFFFFu}) {
    const hobflops::PoolPairs pairs{hw};
    const int64_t last = ((int64_t)hw - 1) / 2 / ahead * ahead;  // the last step's first pair
    int64_t i = last > 32 ? last - 32 : 0;
    int steps = 0;
    for (uint32_t p = (uint32_t)i; pairs.more(p) && steps < 10; p += ahead, i += ahead, ++steps)
      for (uint32_t k = 0; k < ahead; ++k)
        for (uint32_t r = 0; r < 2; ++r) {
          const int64_t pos = 2 * (i + k) + r;
          if (pairs.have(p + k, r) != (pos < hw) || pairs.at(p + k, r) != (pos < hw ? pos : hw - 1))
            return printf("HW %u pair %lld\n", hw, (long long)(i + k)), 1;
        }
    if (i != last + ahead) return printf("HW %u: the walk ends at pair %lld\n", hw, (long long)i), 1;
  }
  return 0;
}
"""


def test_walk_of_the_largest_maps(tmp_path):
    src, exe = tmp_path / "pairs.hip", tmp_path / "pairs"
    src.write_text(SRC)
    r = subprocess.run([build.HIPCC, "-std=c++17", "--cuda-host-only", "-I",
                        os.path.join(build.HERE, "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
