"""Checks of the built library's own gfx950 code that no run can make: what the
compiler did with the inline assembly of the ring loads, whose operands and
wait states it does not look into.  (CPU: the code is disassembled.)"""
import os
import re
import subprocess

import pytest

from paper_1904_07778_amd import xeng

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
LDS_LOAD = re.compile(r"(buffer_load_dword(x4)?|global_load_lds_dword(x4)?)\b")


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """Instruction lists ("opcode operands") by kernel symbol, of the units that hold ring loads."""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    d = tmp_path_factory.mktemp("code")
    lib = d / "libxeng.so"
    os.symlink(xeng.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib.name], cwd=d, check=True, capture_output=True)
    kernels = {}
    for name in sorted(os.listdir(d)):
        if "amdgcn" not in name:
            continue
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", name], cwd=d, check=True, capture_output=True,
                              text=True).stdout
        body = None
        for line in text.splitlines():
            if line.endswith(">:"):
                body = kernels.setdefault(line.split("<", 1)[1][:-2], [])
            elif body is not None and line[:1].isspace():
                body.append(line.split("//")[0].strip())
    kernels = {k: v for k, v in kernels.items() if any(" lds" in i or "load_lds" in i for i in v)}
    assert len(kernels) > 40
    return kernels


def test_row_count_clamp_keeps_its_limit(code):
    """s_max then s_min into one register: the minimum's other operand must not
    be that register too (the upper limit would be lost, and the byte count of
    a stage, rows times the row stride, wraps at 4 GiB)."""
    bad = [k for k, body in code.items() if any(re.fullmatch(r"s_min_i32 (s\d+), \1, \1", i) for i in body)]
    assert not bad, bad


def registers(operand):
    m = re.fullmatch(r"s(\d+)|s\[(\d+):(\d+)\]", operand)
    if not m:
        return []
    return [int(m[1])] if m[1] else list(range(int(m[2]), int(m[3]) + 1))


def too_close(body):
    """LDS loads (index, instruction) that follow a write of M0, or a vector
    instruction's write of a scalar register they read, by fewer wait states
    than CDNA asks for: one after the M0 write, five after the vector write."""
    now, m0, written, bad = 0, -100, {}, []
    for at, ins in enumerate(body):
        op, _, rest = ins.partition(" ")
        operands = [o.strip() for o in rest.split(",")]
        if LDS_LOAD.match(ins) and (op.startswith("global") or ins.endswith("lds")):
            last = max([written.get(r, -100) for o in operands for r in registers(o.split(" ")[0])], default=-100)
            if now - m0 - 1 < 1 or now - last - 1 < 5:
                bad.append((at, ins))
        if op.startswith("s_") and operands[0] == "m0":
            m0 = now
        if op.startswith("v_"):
            for o in operands[:2]:
                for r in registers(o):
                    written[r] = now
        now += int(operands[0], 0) + 1 if op == "s_nop" else 1
    return bad


def test_hazard_rule_on_known_sequences():
    load = "buffer_load_dwordx4 v1, s[4:7], 0 offen lds"
    m0 = "s_mov_b32 m0, s9"
    assert too_close([m0, load]) and not too_close([m0, "s_nop 0", load])
    rfl = "v_readfirstlane_b32 s6, v3"
    assert too_close([rfl, m0, "s_nop 2", load]) and not too_close([rfl, m0, "s_nop 3", load])
    assert not too_close(["v_readfirstlane_b32 s8, v3", m0, "s_nop 0", load])
    assert too_close([m0, "global_load_lds_dwordx4 v[2:3], off"])


def test_ring_loads_keep_their_wait_states(code):
    """The compiler inserts no wait states for loads inside inline assembly."""
    bad = {k: len(b) for k, b in ((k, too_close(body)) for k, body in code.items()) if b}
    assert not bad, bad
