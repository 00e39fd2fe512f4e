"""tests/native/plan_probe.cpp, built on first use and bound with ctypes."""

import ctypes
import os
import subprocess
import tempfile

import paper_2408_09662_amd as xg
from paper_2408_09662_amd import build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
_lib = None


def lib():
    global _lib
    if _lib is None:
        so = os.path.join(tempfile.mkdtemp(prefix="xg_probe"), "plan_probe.so")
        libdir = os.path.dirname(xg._abi.LIB_PATH)
        rocm = os.path.dirname(os.path.dirname(build.HIPCC))
        subprocess.run(["g++", "-std=c++17", "-O1", "-fPIC", "-shared", "-D__HIP_PLATFORM_AMD__",
                        "-I", os.path.join(rocm, "include"), "-I", os.path.join(ROOT, "include"),
                        "-I", os.path.join(libdir, "csrc"), os.path.join(ROOT, "tests", "native", "plan_probe.cpp"),
                        "-o", so, "-L", libdir, "-l:libxg.so", f"-Wl,-rpath,{libdir}"], check=True)
        xg.lib()  # (libxg.so is in the process before what links against it)
        _lib = ctypes.CDLL(so)
    return _lib


def batch_source(programs, path):
    arr = (ctypes.c_void_p * len(programs))(*[p._h.value for p in programs])
    xg._abi.check(lib().probe_batch_source(arr, len(programs), os.fsencode(path)))
    return open(path).read()


def few(p, mode, n):
    return bool(lib().probe_few(p._h, mode, ctypes.c_longlong(n)))


def loaded(p, mode, few):
    return lib().probe_loaded(p._h, mode, int(few))


def compiled(p, mode, few):
    return bool(lib().probe_compiled(p._h, mode, int(few)))


def spoil_few(p, mode):
    lib().probe_spoil_few(p._h, mode)


def code(p, mode, n):
    """(hash of the sources, phases) of the plan that n instances run."""
    f = lib().probe_code
    f.restype = ctypes.c_ulonglong
    phases = ctypes.c_int()
    return f(p._h, mode, ctypes.c_longlong(n), ctypes.byref(phases)), phases.value


def candidates(p, mode, n):
    """[(hash of the sources, whether it is the library's)] of the tuning candidates."""
    h, l = (ctypes.c_ulonglong * 100)(), (ctypes.c_int * 100)()
    k = lib().probe_candidates(p._h, mode, ctypes.c_longlong(n), h, l, 100)
    assert 0 < k <= 100
    return [(h[i], bool(l[i])) for i in range(k)]


def batch_candidates(programs, ns):
    """{workgroup size: hash of the source} of the batch autotuner's candidates."""
    k = len(programs)
    arr, na = (ctypes.c_void_p * k)(*[p._h.value for p in programs]), (ctypes.c_int64 * k)(*ns)
    block, h = (ctypes.c_int * 8)(), (ctypes.c_ulonglong * 8)()
    return {block[i]: h[i] for i in range(lib().probe_batch_candidates(arr, k, na, block, h))}


def batch_grid(tiles, cost, resident, cus):
    k = len(tiles)
    f = lib().probe_batch_grid
    f.restype = ctypes.c_longlong
    return f(k, (ctypes.c_int64 * k)(*tiles), (ctypes.c_int64 * k)(*cost), ctypes.c_longlong(resident),
             ctypes.c_longlong(cus))
