"""The direct global -> LDS loads of gemm.hip in the code that is built: the
compiler adds no wait states around instructions inside inline assembly, so the
ones gfx950 asks for have to be there by themselves.

  * M0 (the loads' LDS address), written by a scalar instruction, is not read by
    the very next instruction: at least one lies between;
  * a scalar base written by a vector instruction (v_readfirstlane and the like)
    is read five instructions later at the earliest.

The code is read in its linear order, label by label (CPU only: it is compiled
to assembly, not run).
"""
import re
import subprocess

import pytest

from paper_2410_12168_amd import build


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    out = tmp_path_factory.mktemp("asm") / "gemm.s"
    flags = [f for f in build.COMMON if f != "-fPIC"]
    r = subprocess.run([build.HIPCC] + flags + build.DEVICE + build.PER_FILE["gemm.hip"] +
                       ["-S", "--cuda-device-only", f"{build.CSRC}/gemm.hip", "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    instructions = []  # (line number, opcode, operands)
    for n, line in enumerate(out.read_text().splitlines(), 1):
        s = line.split(";")[0].strip()
        if s and not s.startswith((".", "#")) and not s.endswith(":"):
            op, _, rest = s.partition(" ")
            instructions.append((n, op, [a.strip() for a in rest.split(",")]))
    return instructions


def sgprs(operand):
    m = re.match(r"s\[(\d+):(\d+)\]|s(\d+)\b", operand)
    if not m:
        return set()
    return set(range(int(m[1]), int(m[2]) + 1)) if m[1] else {int(m[3])}


def wait_states(op, args):
    return int(args[0], 0) + 1 if op == "s_nop" else 1


def violations(code):
    loads, m0, base = 0, [], []
    for i, (n, op, args) in enumerate(code):
        if not op.startswith("global_load_lds"):
            continue
        loads += 1
        regs = sgprs(args[1])
        waited = 0
        for _, o, a in reversed(code[max(0, i - 5):i]):
            if waited < 1 and o.startswith("s_") and a[0] == "m0":
                m0.append(n)
            if waited < 5 and o.startswith("v_") and sgprs(a[0]) & regs:
                base.append(n)
            waited += wait_states(o, a)
    return loads, m0, base


def test_direct_loads_have_their_wait_states(code):
    loads, m0, base = violations(code)
    assert loads > 100
    assert not m0, f"M0 read right after its write, lines {m0[:10]} ({len(m0)})"
    assert not base, f"scalar base read too soon after a vector write, lines {base[:10]}"


def test_the_check_sees_both():
    s = [(1, "s_mov_b32", ["m0", "s4"]), (2, "global_load_lds_dwordx4", ["v1", "s[2:3]"]),
         (3, "v_readfirstlane_b32", ["s3", "v0"]), (4, "s_mov_b32", ["m0", "s4"]),
         (5, "s_nop", ["0"]), (6, "global_load_lds_dwordx4", ["v1", "s[2:3]"])]
    assert violations(s) == (2, [2], [6])
