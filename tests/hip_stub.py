"""Runs Python that drives libxeng.so on a stand-in for the HIP runtime
(hip_stub.cpp): what its host code decides, without a GPU."""
import functools
import os
import subprocess
import sys
import tempfile
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
ROCM = os.environ.get("ROCM_PATH", "/opt/rocm")

# What the snippets start from: X the binding, stub the stand-in, and
# call(handle, n_time, dump=False), one xeng_correlate(_dump) on made-up
# addresses.
PRELUDE = """
import ctypes, sys
stub = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
stub.stub_used.restype = ctypes.c_size_t
stub.stub_limit.argtypes = [ctypes.c_size_t]
from paper_1904_07778_amd import xeng as X

def call(handle, n_time, dump=False):
    v = [1 << 32] * len(n_time)
    if dump:
        return X.xeng_correlate_dump(handle, v, list(n_time), [1 << 33] * len(n_time))
    X.xeng_correlate(handle, v, list(n_time))
"""


@functools.lru_cache(maxsize=None)
def _library():
    out = os.path.join(tempfile.mkdtemp(prefix="hip_stub_"), "hip_stub.so")
    cmd = ["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{ROCM}/include",
           os.path.join(ROOT, "tests", "hip_stub.cpp"), "-o", out]
    try:
        subprocess.run(cmd, check=True, capture_output=True, text=True)
    except FileNotFoundError:
        pytest.skip("no g++")
    return out


def run(snippet):
    """(standard output lines, the library's trace lines) of the snippet."""
    env = dict(os.environ, XENG_TRACE="1")
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(snippet), _library()], cwd=ROOT, env=env,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-3000:]
    return r.stdout.split("\n")[:-1], [l for l in r.stderr.split("\n") if l.startswith("xeng:")]
