"""Host check of the rule that chooses between the two merges of partial results (merge_by_workgroup
of the library's internal header), against measured kernel times: at no measured point is the chosen
form more than 8% slower than the other one. Points: (rows, splits, us by a workgroup per row, us by
a thread per 8 columns), the extremes and both sides of the rule's line at three latent widths and
for the per-head forms."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

LATENT = [  # d_c = 64
          (12, 5, 4.3, 3.2), (12, 7, 4.3, 3.7), (768, 12, 5.1, 6.1), (1536, 12, 6.7, 5.4), (1536, 32, 8.5, 10.9),
          (2400, 20, 10.8, 8.5), (3840, 63, 16.3, 17.9), (12288, 63, 39.7, 33.0),
          # 192
          (12, 63, 5.0, 16.3), (192, 5, 4.8, 4.2), (768, 12, 5.2, 6.0), (1536, 12, 7.9, 6.5), (1536, 32, 10.0, 11.0),
          (2400, 20, 11.3, 9.5), (2400, 63, 20.5, 22.4), (7680, 20, 25.2, 20.1),
          # 512
          (48, 7, 4.7, 4.2), (768, 12, 6.8, 7.1), (1536, 12, 9.6, 8.9), (1536, 63, 30.0, 32.8),
          (2400, 32, 24.9, 27.6), (3840, 12, 17.5, 17.1), (12288, 7, 37.4, 29.2)]
PER_HEAD = [(12, 5, 3.9, 4.5), (768, 5, 4.0, 4.7), (1536, 5, 5.8, 4.8), (1536, 12, 6.4, 8.2), (2400, 20, 10.0, 13.0),
            (3840, 12, 12.6, 9.5), (3840, 32, 15.0, 21.1), (7680, 20, 23.6, 17.6), (7680, 63, 44.4, 69.8),
            (12288, 63, 95.9, 107.1)]


def test_merge_rule(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    calls = "".join(f'  printf("%d ", (int)vmla::merge_by_workgroup({r}, {n}, {str(h).lower()}));\n'
                    for h, pts in ((False, LATENT), (True, PER_HEAD)) for r, n, _, _ in pts)
    src.write_text('#include "vmla_internal.h"\n#include <cstdio>\nint main() {\n' + calls + "}\n")
    build = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-arch=gfx950", "-x", "hip", str(src),
                            "-I", os.path.join(ROOT, "paper_2605_30351_amd", "csrc"),
                            "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    picks = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout.split()
    assert len(picks) == len(LATENT) + len(PER_HEAD)
    bad = [p for p, by_wg in zip(LATENT + PER_HEAD, picks)
           if (p[2] if by_wg == "1" else p[3]) > 1.08 * min(p[2:])]
    assert not bad, bad
