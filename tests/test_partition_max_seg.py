"""Host check of the even split's partial-result count (partition_max_seg of the library's internal
header) against the owners of every row block's first and last unit, over random and edge shapes."""
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
int main() {
  std::mt19937_64 rng(3);
  long bad = 0, checks = 0;
  auto check = [&](int64_t N, int64_t T, int64_t G) {
    G = std::min(G, N * T);
    int want = 1;
    for (int64_t r = 0; r < N; ++r)
      want = std::max(want, attend_owner(r * T + T - 1, N * T, (int)G) - attend_owner(r * T, N * T, (int)G) + 1);
    ++checks;
    if (partition_max_seg(N, T, G) != want && bad++ < 5)
      printf("N=%ld T=%ld G=%ld: %d, not %d\n", (long)N, (long)T, (long)G, partition_max_seg(N, T, G), want);
  };
  for (int64_t N = 1; N <= 24; ++N)
    for (int64_t T = 1; T <= 24; ++T)
      for (int64_t G = 1; G <= N * T; ++G) check(N, T, G);
  for (int it = 0; it < 20000; ++it)
    check(1 + rng() % (it % 2 ? 2000 : 40), 1 + rng() % (it % 3 ? 1100 : 9), 1 + rng() % (it % 5 ? 600 : 1 << 20));
  check(220, 1024, 256);
  check(878, 1024, 256);
  printf("checks %ld bad %ld\n", checks, bad);
  return bad != 0;
}
"""


def test_partition_max_seg(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src, exe = tmp_path / "max_seg.cpp", tmp_path / "max_seg"
    src.write_text(SOURCE)
    build = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-x", "hip", str(src),
                            "-I", os.path.join(ROOT, "paper_2605_30351_amd", "csrc"),
                            "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0 and "bad 0" in run.stdout, run.stdout[-2000:]
