"""Visiting order of wilson_apply's streaming kernel (csrc/canon_order.h),
compiled for the host: a permutation of the sites for extents of one, below
and above the blocks', and inside the lattice at the largest volume that the
library accepts, 2^28 sites, where one extent is 1."""
import os
import subprocess

import pytest

from paper_1005_3043_amd import build

PROGRAM = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
#include "canon_order.h"
static int whole(const mg::CanonOrder &o) {
  const uint32_t V = o.L[0] * o.L[1] * o.L[2] * o.L[3];
  std::vector<char> seen(V, 0);
  for (uint32_t n = 0; n < V; ++n) {
    const uint32_t s = mg::site_at(o, n);
    if (s >= V || seen[s]) return 1;
    seen[s] = 1;
  }
  return 0;
}
static int sampled(const mg::CanonOrder &o) {  // every 61st position and both ends
  const uint64_t V = (uint64_t)o.L[0] * o.L[1] * o.L[2] * o.L[3];
  std::vector<uint32_t> at;
  for (uint64_t n = 0; n < V; n += 61) at.push_back(mg::site_at(o, (uint32_t)n));
  at.push_back(mg::site_at(o, (uint32_t)(V - 1)));
  std::sort(at.begin(), at.end());
  return at.back() >= V || (std::unique(at.begin(), at.end()) != at.end() && (V - 1) % 61 != 0);
}
int main() {
  const int small[][4] = {{1, 1, 1, 1}, {3, 1, 7, 3}, {9, 7, 5, 11}, {5, 17, 1, 2}, {2, 1, 33, 3}, {4, 16, 16, 2},
                          {7, 31, 6, 1}, {1, 3, 2, 5}};
  for (auto &L : small)
    for (int nrhs : {1, 12}) {
      mg::CanonOrder o = mg::canon_order(L, nrhs);
      if (whole(o)) return std::printf("order of %d %d %d %d x%d\n", L[0], L[1], L[2], L[3], nrhs), 1;
    }
  const int large[][4] = {{8, 1, 4096, 8192}, {8, 4096, 1, 8192}, {1, 1, 16384, 16384}, {15, 1, 1, 17895697},
                          {15, 2, 2, 4473924}, {32, 64, 256, 512}};
  for (auto &L : large) {
    std::printf("%d %d %d %d\n", L[0], L[1], L[2], L[3]);
    std::fflush(stdout);
    if (sampled(mg::canon_order(L, 1))) return std::printf("outside the lattice, or twice\n"), 1;
  }
  return 0;
}
"""


def test_order_is_a_permutation(tmp_path):
    if not os.path.exists(build.HIPCC):
        pytest.skip("no hipcc")
    src, exe = tmp_path / "order.cpp", tmp_path / "order"
    src.write_text(PROGRAM)
    subprocess.run([build.HIPCC, "-std=c++17", "-O2", "-x", "hip", "--offload-host-only", "-I", build.CSRC, "-I",
                    build.INCLUDE, str(src), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
