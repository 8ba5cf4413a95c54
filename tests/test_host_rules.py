"""Rules of device code that a host build can run: the order of the singular values is a permutation for any
values, and a word that another launch or other data left behind is no count."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
RANKING = r"""
#include <hip/hip_runtime.h>
#include <cmath>
#include <cstdio>
#include "ranking.hpp"
int main() {
  const double values[] = {NAN, INFINITY, 2.0, 0.0, -0.0, -NAN, -INFINITY};
  enum { N = 5, V = sizeof values / sizeof *values };
  int total = 1, bad = 0;
  for (int i = 0; i < N; ++i) total *= V;
  for (int code = 0; code < total; ++code) {           // every list of N of the values
    double s[N], sorted[N];
    bool seen[N] = {};
    for (int i = 0, c = code; i < N; ++i, c /= V) s[i] = values[c % V];
    for (int a = 0; a < N; ++a) {
      const int rank = glowq::rank_of([&](int b) { return s[b]; }, N, a);
      if (rank >= N || seen[rank]) { ++bad; continue; }
      seen[rank] = true;
      sorted[rank] = s[a];
    }
    for (int i = 0; i + 1 < N && !bad; ++i)            // descending, NaN behind all numbers
      bad += std::isnan(sorted[i]) ? !std::isnan(sorted[i + 1]) : sorted[i] < sorted[i + 1];
  }
  printf("%d of %d lists out of order\n", bad, total);
  return bad != 0;
}
"""
ARRIVALS = r"""
#include <hip/hip_runtime.h>
#include <cstdio>
#include "arrivals.hpp"
int main() {
  const unsigned long long tag = 0x0123456789abcdefull, key = glowq::arrival_key(tag);
  int bad = 0;
  for (unsigned n = 0; n < 1u << glowq::ARRIVAL_BITS; ++n) {
    bad += glowq::arrivals(key | n, key) != n;
    for (int bit = glowq::ARRIVAL_BITS; bit < 64; ++bit) bad += glowq::arrivals((key | n) ^ 1ull << bit, key) != 0;
    for (unsigned other = 2; other < 64; other += 2) bad += glowq::arrivals(glowq::arrival_key(tag + other) | n, key) != 0;
  }
  printf("%d words misread\n", bad);
  return bad != 0;
}
"""


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="hipcc not available")
@pytest.mark.parametrize("main", [RANKING, ARRIVALS], ids=["ranking", "arrivals"])
def test_rule(main, tmp_path):
    src, exe = tmp_path / "rule.hip", str(tmp_path / "rule")
    src.write_text(main)
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_2603_25385_amd", "csrc"),
                    str(src), "-o", exe], check=True, capture_output=True)
    p = subprocess.run([exe], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout + p.stderr
