"""The library's host code on the CPU: libdvl.so over ``fake_hip.cpp`` in a
process of its own (no torch in it, whose libraries bring the real runtime).

A test passes the body of a program that has ``D`` (the binding), ``L`` (the
library), ``H`` (the stand-in runtime), ``np`` and the helpers below.
"""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PROLOGUE = '''
import ctypes as C, sys, types
H = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
H.fake_name.restype = C.c_char_p
sys.modules["torch"] = torch = types.ModuleType("torch")
torch.float32, torch.float16, torch.bfloat16, torch._C = "f32", "f16", "bf16", object()
import importlib.util
import numpy as np
spec = importlib.util.spec_from_file_location("dvl_binding", sys.argv[2])
D = importlib.util.module_from_spec(spec)
spec.loader.exec_module(D)
L = D.lib()
KEEP = []

def ok(status):
    assert status == 0, (status, L.dvl_last_error())

def mem(n=4096):
    """An address that stands for device memory."""
    a = np.zeros(n, np.uint8)
    KEEP.append(a)
    return a.ctypes.data

def build(n, M=4, dtype=0, **opt):
    v, f = C.c_void_p(), (C.c_void_p * M)(*[mem(16)] * M)
    o = D.dvl_build_options(opt.get("tile_steps", 0), opt.get("run_waves", 0), opt.get("entry_cache", 0), opt.get("allocator"))
    ok(L.dvl_build_order_ex(n, mem(16), mem(16), mem(16), mem(16), M, dtype, C.cast(f, C.c_void_p), C.byref(o), None, C.byref(v)))
    return v

def zoom(v, first, last):
    z = C.c_void_p()
    ok(L.dvl_zoom(v, first, last, None, None, C.byref(z)))
    return z

def bins(W, M=4):
    return D.dvl_bins(mem(4 * W), mem(4 * W), mem(4 * M * W), mem(4 * M * W), mem(4 * M * W), mem(4 * M * W), mem(8), mem(4))

def set_tfs(v, M=4, n_tf=256, hi=1.0):
    a = np.linspace(0, 1, n_tf, dtype=np.float32)
    for m in range(M):
        ok(L.dvl_set_tf(v, m, a.ctypes.data, n_tf, 0.0, hi))

def update(v, W, M=4, **kw):
    p = D.params(W, **kw)
    ok(L.dvl_update(v, C.byref(p), C.byref(bins(W, M)), None))

def request(v, W, M=4, n_tf=256, hi=1.0, **kw):
    a = np.tile(np.linspace(0, 1, n_tf, dtype=np.float32), M)
    lo, up = np.zeros(M, np.float32), np.full(M, hi, np.float32)
    KEEP.extend((a, lo, up))
    return D.dvl_request(v, a.ctypes.data, n_tf, lo.ctypes.data, up.ctypes.data, D.params(W, **kw), bins(W, M))

def executor():
    ex = C.c_void_p()
    ok(L.dvl_executor_create(C.byref(ex)))
    return ex

def batch(ex, reqs):
    ok(L.dvl_update_batch(ex, (D.dvl_request * len(reqs))(*reqs), len(reqs), None))

def launched(part=""):
    """(name, grid x, grid y) of the launches whose kernel name holds `part`."""
    out = [(H.fake_name(i).decode(), H.fake_grid(i, 0), H.fake_grid(i, 1)) for i in range(H.fake_launches())]
    return [o for o in out if part in o[0]]
'''


def run(tmp_path, body, timeout=120):
    """Run `body` in a process of its own and return what it printed."""
    lib = os.path.join(ROOT, "paper_2306_11612_amd", "_lib", "libdvl.so")
    if shutil.which("g++") is None or not os.path.exists(lib):
        pytest.skip("needs g++ and the built library")
    stub = os.path.join(str(tmp_path), "fake_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-pthread", os.path.join(HERE, "fake_hip.cpp"), "-o", stub],
                   check=True, capture_output=True, text=True)
    prog = os.path.join(str(tmp_path), "prog.py")
    with open(prog, "w") as fh:
        fh.write(PROLOGUE + textwrap.dedent(body))
    r = subprocess.run([sys.executable, prog, stub, os.path.join(ROOT, "paper_2306_11612_amd", "dvl.py")],
                       capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:], r.stderr[-4000:])
    return r.stdout
