"""The shared-memory sizes of the leading-eigenpair kernels hold every address that the kernels
form: the row solve of the Cholesky-QR loads `width` entries from the start of each of the r rows
of the factor (pitch r + 1), whatever r is.  The sizes are those the launchers pass (the header is
compiled as it is); sizes n and r at which a kernel runs are enumerated."""
import os
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2308_01480_amd", "csrc")

PROGRAM = r"""
#include <cstdio>
#include "eig_layout.h"
int main() {
  int bad = 0;
  for (int n = 1; n <= 256; ++n)
    for (int r = 1; r <= n && r <= 64; ++r) {
      const size_t solve = (size_t)(r - 1) * (r + 1) + (r <= 16 ? 16 : r <= 32 ? 32 : 64);
      // the arrays themselves, in the kernels' order
      const size_t top = (size_t)((n * (n - 1) / 2 + 1) & ~1) + n * (r + 1);
      const size_t wy = (size_t)n * (r + 1) + n * 17 + 16 * (r + 1);
      if (n <= 128) {
        for (int bv = 1; bv <= r; ++bv) {
          const size_t have = ttr::eig_top_lds(n, r, bv) / sizeof(double);
          if (have < top + solve || have < top + 2 * r * (r + 1) + 3 * n * bv) { std::printf("top %d %d %d\n", n, r, bv); ++bad; }
        }
      } else if (r <= 32) {
        const size_t have = ttr::back_wy_lds(n, r) / sizeof(double);
        if (have < wy + solve || have < wy + 2 * r * (r + 1)) { std::printf("wy %d %d\n", n, r); ++bad; }
        if (have * sizeof(double) > 150 * 1024) { std::printf("wy %d %d too large\n", n, r); ++bad; }
      }
    }
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_row_solve_stays_inside(tmp_path):
    src, exe = tmp_path / "layout.cpp", tmp_path / "layout"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", f"-I{CSRC}", str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout[:2000]
