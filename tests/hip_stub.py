"""The library over the host-only HIP runtime of hip_stub.c, in a process of its
own: run(code) executes `code` with V (the binding), lattice() and the launches
and runtime calls recorded so far in its names."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = '''
import ctypes as C, sys
sys.path.insert(0, ROOT)
stub = C.CDLL(STUB, mode=C.RTLD_GLOBAL)   # in front of the library's own runtime
from paper_2409_02964_amd import vanse as V
launches, calls = [], []     # (kernel name, workgroups, arguments), names
fail_launch = lambda name, k: 0
fail_call = lambda name, k: 0

@C.CFUNCTYPE(C.c_int, C.c_char_p, C.c_uint, C.POINTER(C.c_void_p))
def on_launch(name, blocks, args):
    launches.append((name.decode(), blocks, args))
    return int(fail_launch(launches[-1][0], len(launches)))

@C.CFUNCTYPE(C.c_int, C.c_char_p)
def on_call(name):
    calls.append(name.decode())
    return int(fail_call(calls[-1], len(calls)))

C.c_void_p.in_dll(stub, "stub_on_launch").value = C.cast(on_launch, C.c_void_p).value
C.c_void_p.in_dll(stub, "stub_on_call").value = C.cast(on_call, C.c_void_p).value
L = V.lib()
keep = []

def field(n):
    keep.append((C.c_double * n)())
    return C.cast(keep[-1], C.c_void_p)

def lattice(nx, ny, precision="f32", bc_x="periodic", bc_y="periodic", **has):
    """A lattice that is ready to step (the kernels that would fill it do nothing)."""
    d = V.Desc(nx, ny, V.PRECISION[precision], V.BC[bc_x], V.BC[bc_y], *[int(k in has) for k in
               ("force_field", "drag", "mask", "dynamic_phi")])
    n = C.c_size_t()
    V.check(L.vanse_workspace_bytes(C.byref(d), C.byref(n)))
    keep.append((C.c_char * (n.value + 256))())
    h = C.c_void_p()
    base = (C.addressof(keep[-1]) + 255) // 256 * 256
    V.check(L.vanse_create(C.byref(d), C.c_void_p(base), n.value, C.byref(h)))
    r = V.Rates(1.0, 1.2, 1.2, 1.2, 1.2)
    V.check(L.vanse_set_params(h, 0.5, C.byref(r)))
    return h

def ready(h, nx, ny):
    V.check(L.vanse_set_void_fraction(h, field(nx * ny), None))
    V.check(L.vanse_init_equilibrium(h, 1.0, 0.0, 0.0, None))
    launches.clear()
    calls.clear()
    return h
'''


def run(tmp_path, code):
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("gcc not available")
    stub = str(tmp_path / "libhip_stub.so")
    subprocess.run([cc, "-std=c99", "-O1", "-shared", "-fPIC", "-o", stub, os.path.join(HERE, "hip_stub.c")],
                   check=True, timeout=120)
    r = subprocess.run([sys.executable, "-c", f"ROOT = {ROOT!r}\nSTUB = {stub!r}\n" + PRELUDE + code],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
    return r.stdout
