"""What the column-split kernel must keep around its loads to LDS, read from the assembly that its source compiles to.

Wait states that software owes the hardware around inline assembly, where the compiler inserts none: one between a
scalar write of M0 and a load that writes LDS (M0 is its LDS address); five between a vector instruction that writes a
scalar register and a vector-memory access that reads it."""
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


@pytest.fixture(scope="module")
def assembly(tmp_path_factory):
    if shutil.which(build.HIPCC) is None:
        pytest.skip("needs hipcc")
    out = str(tmp_path_factory.mktemp("asm") / "coop.s")
    cmd = [build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", SOURCE, "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    return open(out).read()


def test_loads_to_lds_have_their_wait_states(assembly):
    loads, complaints = missing_wait_states(assembly)
    assert loads > 0
    assert not complaints, f"{len(complaints)} of {loads} loads: {complaints[:3]}"


def test_one_chunk_of_q_at_most_stands_before_the_first_k_and_v(assembly):
    # a compute unit's loads return in order: what the upper row wave issues before the first barrier delays the first tile
    kernels = re.findall(r"^(_ZN4leet21fwd_16bit_coop_kernelILi(\d+)E\w*):(.*?)^\.Lfunc_end", assembly, flags=re.S | re.M)
    walks = [(int(d), body) for _, d, body in kernels if "global_load_lds" in body]
    assert len(walks) == 12
    for d, body in walks:
        assert body.split("s_barrier")[0].count("global_load_lds") <= d // 16
