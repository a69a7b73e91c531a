"""What the library launches, on a machine without a GPU: a child process loads
tests/launch_shim.c in the HIP runtime's place and then libpfresample, runs
the given code against it and returns the launches it recorded.  Pointers are
never followed on the host, so any aligned number stands for device memory."""
import json
import os
import re
import shutil
import subprocess
import sys
import tempfile

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

needs_shim = pytest.mark.skipif(
    shutil.which("gcc") is None or shutil.which("c++filt") is None,
    reason="gcc or c++filt not installed")

PRELUDE = """
import ctypes, json, sys, threading
sys.path.insert(0, {root!r})
shim = ctypes.CDLL({shim!r}, ctypes.RTLD_GLOBAL)
from paper_1301_4019_amd import _lib
_lib.TUNING_PATH = "/nonexistent"
lib = _lib.open_library(_lib.LIB_PATH)
RNG = _lib.Rng(1, 0, 0, None)
def seg(n, filters=1, offsets=None, max_len=0):
    return _lib.Segments(n, filters, offsets, max_len)
GB = 1 << 30
def launches():
    buf, out = ctypes.create_string_buffer(1024), []
    for i in range(shim.shim_count()):
        shim.shim_launch(i, buf, 1024)
        t, grid, block, stream, name = buf.value.decode().split(" ", 4)
        out.append([int(t), int(grid), int(block), int(stream), name])
    shim.shim_clear()
    return out
"""


def run(code):
    """The JSON value that `code` leaves in `result` (kernel names demangled
    where a launch list is returned)."""
    with tempfile.TemporaryDirectory() as tmp:
        shim = os.path.join(tmp, "launch_shim.so")
        subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-pthread", "-o", shim,
                        os.path.join(ROOT, "tests", "launch_shim.c")], check=True)
        prog = PRELUDE.format(root=ROOT, shim=shim) + code + "\nprint(json.dumps(result))\n"
        res = subprocess.run([sys.executable, "-c", prog], capture_output=True, text=True,
                             timeout=120)
    assert res.returncode == 0, res.stderr[-4000:]
    text = subprocess.run(["c++filt"], input=res.stdout.splitlines()[-1], capture_output=True,
                          text=True, check=True).stdout
    return json.loads(text)


def kernel(launch):
    """The bare name of a launch's kernel."""
    return re.search(r"k_\w+", launch[4]).group(0)
