"""Which bytes of a pruned column the kernels for few output blocks clear: their own arithmetic (csrc/zero_cols.h),
built for the host.  With every weight of a layer pruned any M is few output blocks, and 4 M bytes do not fit an
int (CPU)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <cstdio>
#include <initializer_list>
#include "zero_cols.h"
using namespace twg;
static int fails = 0;
static void check(bool ok, int M, int ES, int i) {
  if (!ok && ++fails < 10) std::printf("M %d, %d bytes an element, chunk %d\n", M, ES, i);
}
int main() {
  for (int ES : {1, 4})
    for (int M : {1, 3, 15, 16, 17, 255, 4096, (1 << 29) - 16, 1 << 29, (1 << 29) + 1, 1 << 30, 2147483632}) {
      const int64_t bytes = (int64_t)M * ES;
      const int chunks = zero_chunks(bytes);
      check(chunks > 0 && (int64_t)chunks * 16 >= bytes && ((int64_t)chunks - 1) * 16 < bytes, M, ES, -1);
      // the first and the last chunks of a column, and of the columns behind it where a workgroup takes several
      for (int z = 0; z < (chunks < 512 ? 3 : 1); ++z)
        for (int64_t c = 0; c < chunks; c = c == 2 && chunks > 6 ? chunks - 3 : c + 1) {
          const int i = (int)(z * (int64_t)chunks + c);
          const ZeroChunk x = zero_chunk(i, chunks);
          check(x.column == z && x.at == c * 16 && x.at < bytes, M, ES, i);
        }
    }
  std::printf("fails=%d\n", fails);
  return fails != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_chunks_of_pruned_columns(tmp_path):
    src, exe = tmp_path / "driver.cpp", tmp_path / "driver"
    src.write_text(DRIVER)
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2402_10876_amd", "csrc"), str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "fails=0" in r.stdout, r.stdout[-2000:]
