"""Wait states that software owes the hardware around inline assembly, where the compiler inserts none: read from the
assembly that the library's own sources compile to.

Before a load that writes LDS (its LDS address is M0): one wait state after a scalar write of M0.  Before any
vector-memory access: five after a vector instruction wrote a scalar register that it reads."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2501_02573_amd import build

SOURCE = os.path.join(build.CSRC, "leet_fwd_16bit_coop.hip")


def scalar_registers(text):
    """Numbers of the scalar registers named in an operand list."""
    regs = set()
    for lo, hi in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        regs |= set(range(int(lo), int(hi) + 1))
    return regs | {int(n) for n in re.findall(r"\bs(\d+)\b", text)}


def missing_wait_states(assembly):
    """(loads to LDS that were looked at, complaints)"""
    code = []   # (mnemonic, operands), in order; labels and directives left out
    for line in assembly.splitlines():
        line = line.split(";")[0].strip()
        if line and not line.endswith(":") and line[0] != ".":
            name, _, operands = line.partition(" ")
            code.append((name, operands.strip()))
    loads, complaints = 0, []
    for i, (name, operands) in enumerate(code):
        if not name.startswith("global_load_lds") and not (name.startswith("buffer_load") and "lds" in operands.split()):
            continue
        loads += 1
        reads, states = scalar_registers(operands), 0
        for before, ops in reversed(code[max(0, i - 8):i]):
            written = ops.split(",")[0]
            if states < 1 and before.startswith("s_") and written.strip() == "m0":
                complaints.append(f"{states} wait states between '{before} {ops}' and '{name} {operands}'")
            if states < 5 and before.startswith("v_") and scalar_registers(written) & reads:
                complaints.append(f"{states} wait states between '{before} {ops}' and '{name} {operands}'")
            states += int(ops) + 1 if before == "s_nop" else 1
    return loads, complaints


@pytest.mark.parametrize("code, bad", [
    ("s_mov_b32 m0, s4\nglobal_load_lds_dwordx4 v1, s[2:3]", 1),
    ("s_mov_b32 m0, s4\ns_nop 0\nglobal_load_lds_dwordx4 v1, s[2:3]", 0),
    ("v_readfirstlane_b32 s2, v7\ns_mov_b32 m0, s4\ns_nop 2\nglobal_load_lds_dwordx4 v1, s[2:3]", 1),
    ("v_readfirstlane_b32 s2, v7\ns_mov_b32 m0, s4\ns_nop 3\nglobal_load_lds_dwordx4 v1, s[2:3]", 0),
    ("v_readfirstlane_b32 s4, v7\ns_mov_b32 m0, s4\ns_nop 0\nglobal_load_lds_dwordx4 v1, s[2:3]", 0),
])
def test_the_reading_itself(code, bad):
    loads, complaints = missing_wait_states(code)
    assert loads == 1 and len(complaints) == bad


@pytest.mark.skipif(shutil.which(build.HIPCC) is None, reason="needs hipcc")
def test_loads_to_lds_have_their_wait_states(tmp_path):
    out = str(tmp_path / "coop.s")
    cmd = [build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", SOURCE, "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    loads, complaints = missing_wait_states(open(out).read())
    assert loads > 0
    assert not complaints, f"{len(complaints)} of {loads} loads: {complaints[:3]}"
