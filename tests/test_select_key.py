"""The order of a query's candidates (msac asc, count desc, sample asc,
solution asc) and the place of a key in a list, in the code the kernels use,
compiled for the host.  A generalised P3P sample has up to eight solutions, so
the sample and the solution must tell keys apart for j = 0..7; and the places of
n keys must be 0..n-1 even if keys should be equal in everything, as each place
is written by the key that has it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

DRIVER = r"""
#include <hip/hip_runtime.h>
#include <algorithm>
#include <cstdio>
#include <random>
#include <tuple>
#include <vector>
#include "select_key.h"
using namespace imloc;

int main() {
  int fails = 0;
  // strictly rising over (h, j)
  for (long long h0 : {0ll, 1ll, 1000003ll, 1ll << 40}) {
    long long last = -1;
    for (long long h = h0; h < h0 + 4; ++h)
      for (int j = 0; j < 8; ++j) {
        const long long o = hj_order(h, j);
        if (!(o > last)) { std::printf("order of (%lld, %d)\n", h, j); ++fails; }
        last = o;
      }
  }
  // places: a permutation, the one of a stable sort by (ms, -cnt, h, j)
  std::mt19937 g(7);
  for (int n : {1, 2, 7, 8, 31, 32, 64}) {
    for (int form = 0; form < 4; ++form) {
      std::vector<Key> k(n);
      std::vector<std::tuple<double, int, long long, int>> t(n);
      for (int e = 0; e < n; ++e) {
        const long long h = form == 3 ? 5 : g() % 3;
        const int j = form == 3 ? 2 : g() % 8;
        const double ms = form == 0 ? (double)(g() % 4) : 1.5;
        const int cnt = form <= 1 ? (int)(g() % 3) : 3;
        k[e] = Key{ms, hj_order(h, j), cnt, e};
        t[e] = std::make_tuple(ms, -cnt, h, j);
      }
      std::vector<int> order(n);
      for (int e = 0; e < n; ++e) order[e] = e;
      std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return t[a] < t[b]; });
      for (int p = 0; p < n; ++p)
        if (key_place(k.data(), n, order[p]) != p) { std::printf("n %d form %d place %d\n", n, form, p); ++fails; }
    }
  }
  std::printf("%d failure(s)\n", fails);
  return fails != 0;
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not available")
def test_order_and_places(tmp_path):
    src, exe = str(tmp_path / "driver.hip"), str(tmp_path / "driver")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.run([HIPCC, "-O1", "-std=c++17", "--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", "-I", os.path.join(ROOT, "paper_2601_04185_amd", "csrc"), src, "-o", exe],
                   check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failure(s)" in r.stdout, r.stdout + r.stderr
    shutil.rmtree(str(tmp_path), ignore_errors=True)
