"""How the weight gradient deals k-steps to workgroups (csrc/wgrad_deal.h), compiled for the host: what the kernel takes for granted."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include "wgrad_deal.h"
#include <stdio.h>
#include <random>

int main() {
  std::mt19937_64 rng(1);
  auto real = [&](double lo, double hi) { return std::uniform_real_distribution<double>(lo, hi)(rng); };
  auto whole = [&](int lo, int hi) { return (int)(lo + rng() % (uint64_t)(hi - lo + 1)); };
  long dealt = 0, several = 0;
  for (int n = 0; n < 400000; n++) {
    const int members = whole(2, sste::DEAL_MEMBERS), parts = whole(members + 1, sste::DEAL_PARTS), groups = 256 / parts;
    const int64_t steps = whole(16, n % 2 ? 64 : 1024);
    sste::WgradDeal d;
    if (!sste::deal_group(d, real(1.5, 8.0), real(0.25, 0.75), steps, members, parts, groups)) continue;
    dealt++;
    if (d.members != members || d.parts != parts || d.groups != groups || d.bound[0] != 0 || d.bound[parts] != members * steps) return printf("bounds of problem %d\n", n), 1;
    int64_t done[sste::DEAL_MEMBERS] = {};
    int planes[sste::DEAL_MEMBERS] = {};
    for (int c = 0; c < parts; c++) {             // as k_wgrad_gemm walks it
      int64_t at = d.bound[c];
      if (at >= d.bound[c + 1]) return printf("part %d of problem %d has nothing to do\n", c, n), 1;
      several += (d.bound[c + 1] - 1) / steps != at / steps;
      while (at < d.bound[c + 1]) {
        const int m = (int)(at / steps), plane = c - d.first[m];
        const int64_t end = (m + 1) * steps < d.bound[c + 1] ? (m + 1) * steps : d.bound[c + 1];
        if (plane != planes[m]++ || plane >= (int)((d.segments >> (4 * m)) & 15u) || plane >= sste::most_segments(d)) return printf("plane %d of member %d, problem %d\n", plane, m, n), 1;
        if (at != m * steps + done[m] || end - at < sste::DEAL_SHORTEST) return printf("segment at %ld of problem %d\n", (long)at, n), 1;
        done[m] += end - at;
        at = end;
      }
    }
    for (int m = 0; m < members; m++)
      if (done[m] != steps || planes[m] != (int)((d.segments >> (4 * m)) & 15u)) return printf("member %d of problem %d\n", m, n), 1;
  }
  printf("%ld dealt, %ld parts in two members\n", dealt, several);
  return dealt < 100000 || several < 100000;
}
"""


def test_every_dealt_segment_has_its_plane(tmp_path):
    gxx = os.environ.get("CXX", "g++")
    if not shutil.which(gxx):
        pytest.skip("no host compiler")
    (tmp_path / "deal.cpp").write_text(DRIVER)
    exe = str(tmp_path / "deal")
    res = subprocess.run([gxx, "-O2", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "paper_2409_09099_amd", "csrc"), str(tmp_path / "deal.cpp"), "-o", exe],
                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert res.returncode == 0, res.stdout
    run = subprocess.run([exe], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=100)
    assert run.returncode == 0, run.stdout
