"""The launch of the materialised Omega: for every row count that memory can hold and every column
count, all rows are covered, the launch counts fewer than 2^32 threads (the runtime's limit), and a
work-group's items fit in the 32 bits that it numbers them with."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2308_01480_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "common.h"
int main() {
  int bad = 0;
  const int cols[] = {1, 8, 9, 17, 40, 48, 64, 136, 1024, 1025, 1032, 2040, 2048, 2049, 4096, 100000};
  for (int c : cols)
    for (int64_t nrows = 1; nrows <= (int64_t(1) << 36) / c; nrows = nrows * 17 / 16 + 1)
      for (int64_t n = nrows; n <= nrows + 1; ++n) {
        const int64_t rows = ttr::omega_rows_per_group(n, c), blocks = (n + rows - 1) / rows;
        if (rows < 1 || blocks * 256 >= (int64_t(1) << 32) || blocks * rows < n ||
            rows * ((c + 7) / 8) >= (int64_t(1) << 31)) {
          std::printf("%lld rows of %d: %lld per group\n", (long long)n, c, (long long)rows);
          ++bad;
        }
      }
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_launch_fits(tmp_path):
    src, exe = tmp_path / "grid.cpp", tmp_path / "grid"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[:2000]
