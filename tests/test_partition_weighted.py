"""Host check of the decision to take the weighted split (weighted_split_fits of the library's
internal header): a call's workspace holds the partial-result slots that the shape's neediest window
takes, and for every window of the shape, the partly filled ones among them, a call that may take the
weighted split has no empty share, covers every unit, and leaves no more partial results per row
block than there are slots, under random and extreme weights. (An empty share inside a row block
writes no partial result, but the merges count it.)"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "vmla_internal.h"
#include <algorithm>
#include <cstdio>
#include <random>
using namespace vmla;
std::mt19937_64 rng(5);
long bad = 0, on = 0, off = 0;

// start of share k, by integer division
int64_t start(const uint32_t* w, int G, int64_t U, int k) {
  return (int64_t)((__int128)U * bal_cum(w, k) / bal_cum(w, G));
}

void check(int hw, int window, int chunk, int RB, int batch, int bn, int n_wg) {
  int n_seg = 1;
  for (int f = chunk; f <= window; ++f)
    n_seg = std::max(n_seg, make_partition(64, RB, bn, 256, batch, (int64_t)f * hw, n_wg).max_seg);
  for (int f = chunk; f <= window; ++f) {
    const Partition p = make_partition(64, RB, bn, 256, batch, (int64_t)f * hw, n_wg);
    if (!weighted_split_fits(p, n_seg)) { ++off; continue; }
    ++on;
    for (int it = 0; it < 40; ++it) {
      uint32_t w[8];
      for (int x = 0; x < 8; ++x)
        w[x] = it % 4 == 0 ? kBalOne - 26 + rng() % 53 : it % 4 == 1 ? (rng() % 2 ? kBalMin : kBalMax)
                                                                     : kBalMin + rng() % (kBalMax - kBalMin + 1);
      bool ok = start(w, p.G, p.U, 0) == 0 && start(w, p.G, p.U, p.G) == p.U;
      for (int k = 0; k < p.G; ++k) ok = ok && start(w, p.G, p.U, k) < start(w, p.G, p.U, k + 1);
      // shares that hold a unit of row block r: those that start before its end and end after its start
      for (int64_t r = 0, k = 0; ok && r < (int64_t)batch * RB; ++r) {
        while (start(w, p.G, p.U, k + 1) <= r * p.T) ++k;
        int n = 0;
        for (int64_t j = k; j < p.G && start(w, p.G, p.U, j) < (r + 1) * p.T; ++j) ++n;
        ok = n <= n_seg;
      }
      if (!ok && bad++ < 5)
        printf("hw=%d window=%d frames=%d RB=%d batch=%d wg=%d: G=%d U=%ld T=%d n_seg=%d\n", hw, window, f, RB,
               batch, n_wg, p.G, (long)p.U, p.T, n_seg);
    }
  }
}

int main() {
  check(60, 21, 2, 1, 1, 32, 0);      // one row block: one tile per workgroup while the window fills
  check(1560, 21, 3, 220, 1, 32, 0);  // the Wan chunk
  for (int it = 0; it < 1500; ++it) {
    const int window = 1 + rng() % 24, chunk = 1 + rng() % window;
    const int hw = 1 + rng() % (it % 4 ? 300 : 1600), RB = 1 + rng() % (it % 2 ? 6 : 250);
    check(hw, window, chunk, RB, 1 + rng() % 3, 32, it % 3 ? 0 : 1 + rng() % 300);
  }
  printf("weighted %ld even %ld bad %ld\n", on, off, bad);
  return bad != 0 || on < 500 || off < 500;
}
"""


def test_weighted_split_has_no_empty_share(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src, exe = tmp_path / "weighted.cpp", tmp_path / "weighted"
    src.write_text(SOURCE)
    build = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-x", "hip", str(src),
                            "-I", os.path.join(ROOT, "paper_2605_30351_amd", "csrc"),
                            "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "bad 0" in run.stdout, run.stdout[-2000:]
