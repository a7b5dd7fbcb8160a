"""The launches that a library's host code makes, recorded without a GPU.

`launches(body)` runs the Python source `body` in a process of its own, where
the stand-in runtime of hip_recorder.c takes the HIP calls, and returns what the
body assigns to `out`.  The body finds: `handle3(...)` and `handle2(...)`, an
initialised lattice of libcmlbm or libcmlbm2d over made-up device addresses;
`rec(fail=-1, capture=0, cus=256)`, which forgets the launches so far; and
`seen()`, the launches since as [kernel, grid, block, first two arguments].
"""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = """
import ctypes, json, sys
sys.path.insert(0, {root!r})
R = ctypes.CDLL({lib!r}, mode=ctypes.RTLD_GLOBAL)
from paper_1905_10182_amd import cmlbm as B3, cmlbm2d as B2, cmnn as NN
L3, L2, LN = B3.load_library(), B2.load_library(), NN.load_library()
demangle = ctypes.CDLL("libstdc++.so.6").__cxa_demangle
demangle.restype = ctypes.c_char_p
class Dim(ctypes.Structure):
    _fields_ = [(c, ctypes.c_uint32) for c in "xyz"]
class Launch(ctypes.Structure):
    _fields_ = [("name", ctypes.c_char_p), ("grid", Dim), ("block", Dim), ("arg", ctypes.c_void_p * 2)]
R.rec_get.restype = ctypes.POINTER(Launch)
def rec(fail=-1, capture=0, cus=256):
    R.rec_reset(fail, capture, cus)
def seen():
    rows = []
    for i in range(R.rec_count()):
        l = R.rec_get(i)[0]
        name = demangle(l.name.replace(b"DF16b", b"s"), None, None, None)  # (no BF16 in older demanglers)
        name = name.decode().replace("(anonymous namespace)::", "")
        rows.append([name[name.index("k"):name.index("(")].removeprefix("void "), [l.grid.x, l.grid.y, l.grid.z],
                     l.block.x, l.arg[0], l.arg[1]])
    return rows
A, B, S, F, STREAM = 1 << 44, 2 << 44, 3 << 44, 4 << 44, ctypes.c_void_p(64)
def handle3(nx, ny, nz, nbatch=1, storage="fp64", wall=0, field=0):
    p = B3.make_params(nx=nx, ny=ny, nz=nz, nbatch=nbatch, tau=0.8, rho0=1.0, storage=storage, wall=(0, wall, 0), flags=0)
    pop, scratch = B3.required_bytes(p)
    h = ctypes.c_void_p()
    assert L3.cmlbm_create(ctypes.byref(p), A, pop, B, pop, S, scratch, ctypes.byref(h)) == 0
    if field:
        assert L3.cmlbm_set_force(h, B3.FORCE_FIELD, None, F, B3.FP64 if storage == "fp64" else B3.FP32, None) == 0
    assert L3.cmlbm_init(h, None, None, 0, None) == 0
    return h
def handle2(nx, ny, storage="fp64", field=0):
    p = B2.make_params(nx, ny, storage=storage)
    pop, h = B2.required_bytes(p), ctypes.c_void_p()
    assert L2.cmlbm2d_create(ctypes.byref(p), A, pop, B, pop, ctypes.byref(h)) == 0
    if field:
        assert L2.cmlbm2d_set_force(h, B2.FORCE_FIELD, None, F, B2.FP64 if storage == "fp64" else B2.FP32, None) == 0
    assert L2.cmlbm2d_init(h, None, None, 0, None) == 0
    return h
def time_of(get, h):
    t = ctypes.c_int64()
    assert get(h, ctypes.byref(t)) == 0
    return t.value
rec()
"""

_lib = None


def launches(body):
    global _lib
    if _lib is None:
        import tempfile
        _lib = tempfile.TemporaryDirectory()
        subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-w", os.path.join(HERE, "hip_recorder.c"), "-o",
                        os.path.join(_lib.name, "recorder.so")], check=True)
    prelude = PRELUDE.format(root=os.path.dirname(HERE), lib=os.path.join(_lib.name, "recorder.so"))
    res = subprocess.run([sys.executable, "-c", prelude + body + "\nprint(json.dumps(out))"], capture_output=True,
                         text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]
    return json.loads(res.stdout.splitlines()[-1])
