"""The order of the products' 256 x 256 tiles (csrc/tile_order.h), compiled for the host."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "tile_order.h"
#include <stdio.h>
#include <vector>

int main() {
  for (int m = 1; m <= 420; m++)
    for (int n : {1, 2, 3, 4, 5, 13, 14, 15, 64, 128}) {
      const sste::TileOrder o = sste::tile_order(m, n);
      if (o.runs != 1 && (m < 18 || m * n <= 256)) return printf("%d runs of %d x %d tiles\n", o.runs, m, n), 1;
      std::vector<char> seen(m * n);
      int run_first = 0, last_n = 0;
      for (int k = 0; k < m * n; k++) {
        int tm = -1, tn = -1;
        sste::tile_at(o, k, tm, tn);
        if (tm < 0 || tm >= m || tn < 0 || tn >= n || seen[tm * n + tn]++) return printf("tile %d of %d x %d\n", k, m, n), 1;
        if (tn < last_n) run_first = tm;          // the next run
        last_n = tn;
        if (o.runs > 1 && n > 1 && (tm < run_first || tm >= run_first + (m <= 73 ? 19 : 14))) return printf("too long a run of %d x %d tiles\n", m, n), 1;
      }
    }
  for (long m : {1000L, 100000L, 8000000L}) {     // wide weights: the products stay in 32 bits
    const sste::TileOrder o = sste::tile_order(m, 100);
    int tm, tn;
    sste::tile_at(o, (int)(m * 100 - 1), tm, tn);
    if (tm != m - 1 || tn != 99) return printf("last of %ld x 100 tiles\n", m), 1;
  }
  return 0;
}
"""


def test_every_tile_once_in_runs_of_about_ten(tmp_path):
    gxx = os.environ.get("CXX", "g++")
    if not shutil.which(gxx):
        pytest.skip("no host compiler")
    (tmp_path / "order.cpp").write_text(DRIVER)
    exe = str(tmp_path / "order")
    res = subprocess.run([gxx, "-O1", "-std=c++17", "-Wall", "-ftrapv", "-I", os.path.join(ROOT, "paper_2409_09099_amd", "csrc"), str(tmp_path / "order.cpp"), "-o", exe],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=100)
    assert run.returncode == 0, run.stdout
