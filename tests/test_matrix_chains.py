"""Waits between dependent matrix products in the built code: a product that adds
to the sum of a product of another shape reads it from the registers, and neither
the hardware nor the compiler waits for it (csrc/mfma.h).  The kernels are
compiled to assembly and every such pair has to have five wait states of s_nop
between them, whatever other instructions the compiler put there."""
import os
import re
import subprocess

import pytest

from paper_1904_02033_amd import build

WAIT = 5


def _regs(op):
    """Register names of an operand such as v7, v[4:7] or a[0:3]."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", op)
    if not m:
        return []
    lo = int(m.group(2) or m.group(3))
    return [(m.group(1), r) for r in range(lo, int(m.group(2) or m.group(4)) + 1)]


def mixed_chains(lines):
    """(pairs of products of different shapes in one sum, those that have too few
    wait states of s_nop between them) of one function's assembly."""
    last, nops, pairs, short = {}, 0, 0, []
    for i, line in enumerate(lines):
        t = line.split(";")[0].split()
        if not t or t[0].endswith(":") or t[0].startswith("."):
            continue
        ops = [o.rstrip(",") for o in t[1:]]
        if t[0] == "s_nop":
            nops += int(ops[0]) + 1
        elif t[0].startswith("v_mfma"):
            prev = [last[r] for r in _regs(ops[3]) if r in last and last[r][0] != t[0]]
            pairs += bool(prev)
            if any(nops - n < WAIT for _, n in prev):
                short.append((i, line.strip()))
            for r in _regs(ops[0]):
                last[r] = (t[0], nops)
        elif ops and t[0][:2] in ("v_", "ds", "gl", "bu", "sc"):
            for r in _regs(ops[0]):
                last.pop(r, None)
    return pairs, short


def test_scan():
    mm = ["v_mfma_i32_16x16x64_i8 a[4:7], v[2:5], v[6:9], 0",
          "v_mfma_i32_16x16x32_i8 a[4:7], v[2:3], v[6:7], a[4:7]"]
    for wait, ok in (([], False), (["s_nop 3"], False), (["s_nop 4"], True),
                     (["v_mov_b32_e32 v0, v1"] * 9, False), (["s_nop 0"] * 5, True)):
        pairs, short = mixed_chains([mm[0]] + wait + [mm[1]])
        assert pairs == 1 and (not short) == ok, wait
    assert mixed_chains([mm[0], "v_accvgpr_write_b32 a5, v0", mm[0]])[0] == 0


@pytest.mark.parametrize("source,kernel,mixed", [
    ("kmeans.hip", "k_km_assign", ("Li24E", "Li40E", "Li56E")),
    ("mfma.hip", "k_mac_mfma", ("Li96E",))])
def test_built_chains(tmp_path, source, kernel, mixed):
    out = str(tmp_path / "k.s")
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.check_call([hipcc] + build.FLAGS + ["--cuda-device-only", "-S", "-w",
                                                   os.path.join(build.CSRC, source), "-o", out],
                          stderr=subprocess.DEVNULL)
    names, cur = {}, None
    for line in open(out):
        m = re.match(r"(_Z\w+):", line)
        if m:
            cur = names.setdefault(m.group(1), [])
        elif cur is not None:
            cur.append(line)
    seen = set()
    for name, lines in names.items():
        if kernel not in name:
            continue
        pairs, short = mixed_chains(lines)
        assert not short, (name, short[:3])
        if pairs:
            seen.update(m for m in mixed if m in name)
        assert pairs == 0 or any(m in name for m in mixed), name
    assert seen == set(mixed)
