"""Grids of the device packer's kernels: their own arithmetic (csrc/grid.h), built for the host.  From 2^35 elements on a
weight has more threads than one dimension of a launch takes (CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include <initializer_list>
#include "grid.h"
using namespace twg;
int main() {
  int fails = 0;
  for (uint32_t threads : {128u, 256u, 512u, 1024u})
    for (int shift = 0; shift <= 30; ++shift)
      for (int d = -2; d <= 2; ++d) {
        const uint64_t n = (1ull << shift) + d;
        if (n < 1 || n > 1ull << 30) continue;
        const Grid2 g = grid_of(n, threads);
        const uint64_t all = (uint64_t)g.x * g.y;
        const bool ok = g.x >= 1 && g.y >= 1 && (uint64_t)g.x * threads < 1ull << 32 && all >= n && all - n < g.x && all < 1ull << 32 &&
                        g.y <= 65535 && (n * threads >= 1ull << 32 || (g.x == n && g.y == 1));
        if (!ok && ++fails < 10) std::printf("%llu workgroups of %u: %u x %u\n", (unsigned long long)n, threads, g.x, g.y);
      }
  std::printf("fails=%d\n", fails);
  return fails != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_grids_of_many_workgroups(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2402_10876_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "fails=0" in r.stdout, r.stdout[-2000:]
