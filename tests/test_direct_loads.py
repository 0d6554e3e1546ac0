"""Host check of the generated code around the direct global-to-LDS loads with a scalar base
(lds_dma16_add and lds_dma16_min of csrc/vmla_device.h): no VALU instruction writes a load's scalar
base in the five wait states before it, on any path. The loads are in inline assembly, for which the
compiler does not keep that distance. Compiles the two sources that use them for gfx950, as build.py
does, and reads the assembly."""
import os
import re
import shutil
import subprocess

import pytest

from tests._build_once import _builder

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
WAIT_STATES = 5


def scalar_registers(arg):
    m = re.match(r"s\[(\d+):(\d+)\]$", arg)
    if m:
        return set(range(int(m[1]), int(m[2]) + 1))
    m = re.match(r"s(\d+)$", arg)
    return {int(m[1])} if m else set()


def parse(text):
    """[(op, args)], a label as (None, name); label -> indices of the branches to it."""
    code, sources = [], {}
    for line in text.splitlines():
        t = re.split(r";|//", line)[0].strip()
        if t.endswith(":"):
            code.append((None, t[:-1]))
        elif t and not t.startswith("."):
            op, _, rest = t.partition(" ")
            args = [a.strip().split(" ")[0] for a in rest.split(",")]
            if op.startswith(("s_branch", "s_cbranch")):
                sources.setdefault(args[0], []).append(len(code))
            code.append((op, args))
    return code, sources


def writers(code, sources, at, base, states):
    """VALU writes of `base` within `states` wait states before index `at`, over all paths."""
    bad = []
    while at > 0 and states > 0:
        at -= 1
        op, args = code[at]
        if op is None:
            for src in sources.get(args, ()):
                bad += writers(code, sources, src, base, states - 1)
            continue
        if op in ("s_branch", "s_endpgm", "s_setpc_b64"):
            break
        if op.startswith("v_") and scalar_registers(args[0]) & base:
            bad.append((op, args))
        states -= 1 + (int(args[0]) if op == "s_nop" else 0)
    return bad


def test_scan_finds_a_planted_write():
    load = "global_load_lds_dwordx4 v1, s[4:5]"
    near = "v_readfirstlane_b32 s4, v0\n s_add_u32 m0, s2, s3\n v_add_u32_e32 v1, s6, v2\n " + load
    loop = "L1:\n s_add_u32 m0, s2, s3\n " + load + "\n v_readlane_b32 s5, v9, 1\n s_cbranch_scc1 L1\n"
    far = near.replace("s_add", "s_nop 2\n s_add")
    for text, n in ((near, 1), (loop, 1), (far, 0)):
        code, sources = parse(text)
        at = next(i for i, c in enumerate(code) if c[0] and c[0].startswith("global_load_lds"))
        assert len(writers(code, sources, at, {4, 5}, WAIT_STATES)) == n, text


@pytest.mark.parametrize("source", ["k_attend_wide.hip", "k_dense.hip"])
def test_scalar_bases_are_settled(tmp_path, source):
    build = _builder()
    if shutil.which(build.HIPCC) is None:
        pytest.skip("hipcc not found")
    asm = tmp_path / "out.s"
    r = subprocess.run([build.HIPCC, *build.COMMON, "-x", "hip", "--cuda-device-only", "-S",
                        os.path.join(build.CSRC, source), "-o", str(asm)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    code, sources = parse(asm.read_text())
    loads = 0
    for i, (op, args) in enumerate(code):
        if op == "global_load_lds_dwordx4" and len(args) > 1 and scalar_registers(args[1]):
            loads += 1
            bad = writers(code, sources, i, scalar_registers(args[1]), WAIT_STATES)
            assert not bad, (source, args, bad)
    assert loads >= 24, (source, loads)
