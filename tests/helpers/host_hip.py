"""libu1ml's host side on the CPU: a child interpreter in which the library's
HIP calls go to host_hip.cpp.  The child runs `code` with these names:

  u1          the binding module
  make(spec)  a context (its workspace address is never read)
  ok(status)  asserts U1ML_OK
  launches()  [(kernel name, grid, block, lds, mangled name)] since the last call
  put(x)      leaves x (JSON) for the caller
"""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(os.path.dirname(HERE))

_CHILD = """
import ctypes as C, json, re, sys
H = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_1309_3859_amd import u1ml as u1

class Launch(C.Structure):
    _fields_ = [("name", C.c_char_p), ("grid", C.c_uint32 * 3), ("block", C.c_uint32 * 3), ("lds", C.c_uint64)]

H.host_hip_launches.restype = C.c_size_t
H.host_hip_launch.restype = C.POINTER(Launch)
H.host_hip_launch.argtypes = [C.c_size_t]
L = u1.lib()

def ok(status, ctx=None):
    assert status == 0, (status, L.u1ml_last_error(ctx))

def make(spec):
    h = C.c_void_p()
    ok(L.u1ml_create(C.byref(spec.struct()), C.c_void_p(1 << 40), 1 << 50, None, C.byref(h)))
    H.host_hip_clear()
    return h

def launches():
    v = [H.host_hip_launch(i).contents for i in range(H.host_hip_launches())]
    def name(mangled):  # _ZN4u1ml<length><name>...
        n, rest = re.match(r"_ZN4u1ml([0-9]+)(.*)", mangled).groups()
        return rest[: int(n)]
    out = [(name(l.name.decode()), list(l.grid), list(l.block), l.lds, l.name.decode()) for l in v]
    H.host_hip_clear()
    return out

def put(x):
    print(json.dumps(x), flush=True)
"""


def build(folder) -> str:
    so = os.path.join(str(folder), "libhost_hip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", so, os.path.join(HERE, "host_hip.cpp")],
                   check=True)
    return so


def run(so: str, code: str, timeout: float = 120.0):
    """The values that `code` put, in order; the child's failure is an assertion."""
    r = subprocess.run([sys.executable, "-c", _CHILD + code, so, ROOT], capture_output=True, text=True, timeout=timeout)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
    return [json.loads(x) for x in r.stdout.splitlines()]
