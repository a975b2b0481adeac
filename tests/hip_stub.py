"""The library's host side without a GPU.  run(code) runs `code` in a child process in
which tests/hip_stub.c stands in for the HIP runtime, and returns what it printed.

The code finds `S` (the stub's functions), `L` (the library), `geom(n, off)`, `create(geom,
**settings)` (a handle or the error code), `solve(handle, geom, cycles)` (the error code) and
`kernels()` (the signatures of the kernels launched so far).
"""
import os
import subprocess
import sys

from conftest import ROOT

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = r'''
import ctypes, re, subprocess, sys, types
S = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
from paper_2001_02327_amd import _lib
assert "torch" not in sys.modules
L = _lib.lib()
S.stub_log.restype = ctypes.c_char_p
for f in (S.stub_used, S.stub_queries, S.stub_syncs, S.stub_live): f.restype = ctypes.c_long
S.stub_limit.argtypes = [ctypes.c_long]

def geom(n, off=None, parent=None):
    n = list(n)
    dim = len(n[0])
    return types.SimpleNamespace(dim=dim, n=n, off=off or [(0, 0, 0)], dx0=1.0 / 32, G=1.0, parent=parent)

def create(g, **kw):
    cfg = _lib.make_config(g, **kw)
    h = ctypes.c_void_p()
    rc = L.nested_poisson_create(ctypes.byref(cfg), None, ctypes.byref(h))
    return h if rc == 0 else rc

def solve(h, g, cycles=2):
    k = len(g.n)
    L.nested_poisson_set_fixed_cycles(h, (ctypes.c_int * k)(*[cycles] * k))
    st = _lib.NpStats()
    return L.nested_poisson_solve(h, (ctypes.c_void_p * k)(*[64] * k), 64, ctypes.byref(st))

def kernels():
    names = [l.split() for l in S.stub_log().decode().splitlines()]
    out = subprocess.run(["c++filt"], input="\n".join(l[0] for l in names), capture_output=True, text=True).stdout.splitlines()
    return [re.sub(r"np::|\(anonymous namespace\)::", "", o) for o in out]
'''


def stub():
    """Path of the built stand-in."""
    lib = os.path.join(HERE, "build", "libhip_stub.so")
    src = os.path.join(HERE, "hip_stub.c")
    if not os.path.exists(lib) or os.path.getmtime(lib) < os.path.getmtime(src):
        os.makedirs(os.path.dirname(lib), exist_ok=True)
        tmp = "%s.tmp%x" % (lib, os.getpid())
        subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", tmp, src], check=True)
        os.replace(tmp, lib)
    return lib


def run(code):
    r = subprocess.run([sys.executable, "-c", PRELUDE + code, stub(), ROOT], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout


def run_host_part(source, code, tmp):
    """Compiles the host part of csrc/`source` with `code` behind it (a main()) and runs it."""
    src, exe = os.path.join(tmp, "host_part.hip"), os.path.join(tmp, "host_part")
    with open(src, "w") as fh:
        fh.write('#include "%s"\n%s' % (os.path.join(ROOT, "paper_2001_02327_amd", "csrc", source), code))
    subprocess.run([os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "--offload-host-only", "-c", "-O1", "-std=c++17", "-fPIC",
                    "-o", exe + ".o", src], check=True, capture_output=True)
    # (the device code that the object refers to is left out)
    subprocess.run(["g++", "-o", exe, exe + ".o", stub(), "-Wl,--unresolved-symbols=ignore-all"], check=True, capture_output=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stdout + r.stderr
    return r.stdout
