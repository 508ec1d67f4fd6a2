"""The library's host side on the CPU, over hip_stub.c: a child process calls
the C ABI and gives back what it allocated and launched."""
from __future__ import annotations

import json
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(ROOT, "paper_1908_02464_amd", "libweno_l2is.so")

# `capi`: the binding (its torch is not needed by the calls made here), `L`
# the library, `stub` the stand-in; U and V are device addresses of arrays
PRELUDE = r'''
import ctypes as C, json, subprocess, sys, types
sys.path.insert(0, {root!r})
stub = C.CDLL({stub!r}, mode=C.RTLD_GLOBAL)
stub.stub_log.restype = C.c_char_p
stub.stub_capacity.argtypes = [C.c_size_t]
stub.stub_used.restype = stub.stub_peak.restype = C.c_size_t
torch = sys.modules["torch"] = types.ModuleType("torch")
torch.float64 = None
from paper_1908_02464_amd import capi
L = capi.lib()
U, V = 1 << 56, 1 << 58

def create(shape, dx=0.1, expect=0, stream=None, **kw):
    p = capi.params_default(*shape, dx, **kw)
    h = C.c_void_p()
    rc = L.weno_l2is_create(*shape, dx, 1.4, C.byref(p), C.c_void_p(stream), C.byref(h))
    assert rc == expect, rc
    return h

def log(clear=True):
    """Lines of the log since it was last cleared."""
    s = stub.stub_log().decode().split("\n")[:-1]
    if clear:
        stub.stub_clear()
    return s

def launches():
    """(kernel, grid x, y, z, threads per workgroup), names readable."""
    rows = [r.split()[1:] for r in log() if r.startswith("launch")]
    names = subprocess.run(["c++filt"], input="\n".join(r[0] for r in rows), capture_output=True,
                           text=True).stdout.split("\n")
    return [(n, *map(int, r[1:])) for n, r in zip(names, rows)]
'''


@pytest.fixture(scope="session")
def host_calls(tmp_path_factory):
    """host_calls(code): what `code` assigns to `out`, as JSON."""
    if shutil.which("gcc") is None or shutil.which("c++filt") is None:
        pytest.skip("gcc or c++filt not found")
    if not os.path.exists(LIB):
        pytest.skip("library not built (run __graft_entry__.build())")
    so = str(tmp_path_factory.mktemp("hip") / "libhip_stub.so")
    subprocess.run(["gcc", "-std=c11", "-O1", "-Wall", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "hip_stub.c")],
                   check=True)

    def run(code: str):
        src = PRELUDE.format(root=ROOT, stub=so) + code + "\nprint('OUT ' + json.dumps(out))\n"
        r = subprocess.run([sys.executable, "-c", src], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-3000:]
        return json.loads([l for l in r.stdout.split("\n") if l.startswith("OUT ")][-1][4:])

    return run
