"""Runs a piece of Python in a process of its own where the HIP runtime is tests/native/hip_stub.cpp: nothing is launched, what would be is
recorded.  The piece finds `hac` (the package) and `stub` (the recorder's functions) and prints its answer as JSON."""
import json
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEAD = """
import ctypes as C, json, sys
sys.path.insert(0, {root!r})
import paper_2108_12704_amd as hac
lib, stub = hac.load_library(), C.CDLL({stub!r})
def events():
    out, grid, lds, arg = [], C.c_uint32(), C.c_uint64(), C.c_uint64()
    for i in range(stub.stub_count()):
        what = chr(stub.stub_event(i, C.byref(grid), C.byref(lds), C.byref(arg)))
        out.append((what, grid.value, lds.value, arg.value))
    return out
"""


def run(tmp_path, piece):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no g++")
    so = str(tmp_path / "libhip_stub.so")
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-fPIC", "-shared", "-Wall", os.path.join(ROOT, "tests", "native", "hip_stub.cpp"), "-o", so])
    env = dict(os.environ)
    env["LD_PRELOAD"] = " ".join(filter(None, (so, env.get("LD_PRELOAD"))))
    done = subprocess.run([sys.executable, "-c", HEAD.format(root=ROOT, stub=so) + piece], env=env, capture_output=True, text=True, timeout=300)
    assert done.returncode == 0, done.stderr[-2000:]
    return json.loads(done.stdout.splitlines()[-1])
