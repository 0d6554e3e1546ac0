"""Host check of the rule that sends a dense cache write to the 256 x 256-tile kernel
(dense_write_wide of the library's internal header): every shape of tests/test_gpu_dense_wide.py takes
it, whatever the device's compute units in a wide range, calls of one or two rounds of small tiles and
heads that are not whole 16-byte chunks never do, and the measured calls on both sides of the line
(256 compute units, d_head 128) go where they were faster."""
import os
import shutil
import subprocess

import pytest

from tests.test_gpu_dense_wide import BATCH, CHUNK, CU_COUNTS, GRID_H, GRID_W, SHAPES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_dense_write_rule(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    tokens = CHUNK * GRID_H * GRID_W
    # (batch, tokens, heads, d_head, compute units), wide or not
    points = [((BATCH, tokens, h, dv, cu), 1) for h, dv, _ in SHAPES for cu in CU_COUNTS]
    points += [((4, 4680, 12, 128, 256), 1), ((1, 3120, 16, 128, 256), 1)]
    points += [((1, 1560, 12, 128, 256), 0), ((1, 1, 12, 128, 256), 0), ((1, 512, 12, 128, 256), 0),
               ((1, 2560, 12, 128, 256), 0), ((4, 4680, 32, 68, 256), 0)]
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text('#include "vmla_internal.h"\n#include <cstdio>\nint main() {\n' + "".join(
        '  printf("%d ", (int)vmla::dense_write_wide({}, {}, {}, {}, {}));\n'.format(*p) for p, _ in points) + "}\n")
    build = subprocess.run([hipcc, "-std=c++17", "-O1", "--offload-arch=gfx950", "-x", "hip", str(src),
                            "-I", os.path.join(ROOT, "paper_2605_30351_amd", "csrc"),
                            "-o", str(exe)], capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-2000:]
    got = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60, check=True).stdout.split()
    assert len(got) == len(points)
    bad = [p for (p, want), g in zip(points, got) if int(g) != want]
    assert not bad, bad
