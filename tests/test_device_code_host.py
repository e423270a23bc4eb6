"""Checks of the built library's own gfx950 code that no run can make: what the
compiler did with the inline assembly of the ring loads, whose operands and
wait states it does not look into.  (CPU: the code is disassembled.)"""
import os
import re
import subprocess

import pytest

from paper_1904_07778_amd import xeng

OBJDUMP = os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin", "llvm-objdump")
LDS_LOAD = re.compile(r"\b(buffer_load_dword(?:x4)?|global_load_lds_dword(?:x4)?)\b.*")


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
