"""Runs the library's host side against a recording HIP runtime (host_hip.cpp), in a process of its own."""
import json
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = r'''
import ctypes, json, sys
from ctypes import byref, c_double, c_float, c_int32, c_int64, c_size_t, c_uint32, c_void_p
R = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
R.host_hip_log.restype = ctypes.c_char_p
R.host_hip_used.restype = c_size_t
L = ctypes.CDLL(sys.argv[2])
L.ptycho_last_error.restype = ctypes.c_char_p
L.ptycho_workspace_bytes.restype = c_int64
budget = lambda n: R.host_hip_budget(c_size_t(n))
class Tile(ctypes.Structure):
    _fields_ = [(n, c_int32) for n in "ty0 ty1 tx0 tx1 ey0 ex0 eh ew".split()] + [("grad", c_void_p)]
class State(ctypes.Structure):
    _fields_ = Tile._fields_[:8] + [(n, c_void_p) for n in ("obj", "acc", "grad")]
def context(M, S, capacity):
    h = c_void_p()
    rc = L.ptycho_create(byref(h), M, S, c_double(0.0197), c_double(2.0), c_double(0.1), capacity, None)
    return rc, h
def log():
    out = R.host_hip_log().decode().splitlines()
    R.host_hip_clear()
    return out
def done(**result):
    print("RESULT" + json.dumps(result))
next_address = 1 << 40
def device(nbytes):  # an address range of its own; nothing reads it
    global next_address
    p = next_address
    next_address += (nbytes + 255) // 256 * 256
    return c_void_p(p)
def boxes(H, W, ny, nx, halo):
    for ty in range(ny):
        for tx in range(nx):
            t = (ty * H // ny, (ty + 1) * H // ny, tx * W // nx, (tx + 1) * W // nx)
            ey0, ex0 = max(t[0] - halo, 0), max(t[2] - halo, 0)
            yield t + (ey0, ex0, min(t[1] + halo, H) - ey0, min(t[3] + halo, W) - ex0)
'''


def run(code: str) -> dict:
    """Runs code after the prelude; returns what it passed to done()."""
    import paper_2205_06327_amd as pt
    with tempfile.TemporaryDirectory() as tmp:
        so = os.path.join(tmp, "host_hip.so")
        subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        os.path.join(HERE, "host_hip.cpp"), "-o", so], check=True)
        p = subprocess.run([sys.executable, "-c", PRELUDE + code, so, pt._binding.LIB_PATH], capture_output=True,
                           text=True, timeout=120)
    assert p.returncode == 0, p.stderr[-3000:]
    return json.loads([x for x in p.stdout.splitlines() if x.startswith("RESULT")][-1][6:])
