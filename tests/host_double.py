"""The library over tests/hip_runtime_double.cpp: its host code without a GPU.  In a process of its own, as the stand-in takes
the place of the HIP runtime there: `run(body)` runs the lines of `body` with the names below in a child."""
import functools
import os
import subprocess
import sys
import tempfile
import textwrap

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)

PRELUDE = """
import ctypes as C, sys, types
sys.path.insert(0, %(root)r)
D = C.CDLL(%(double)r, mode=C.RTLD_GLOBAL)          # before the library: its calls to the runtime come here
for f in ("double_in_use", "double_blocks", "double_freed", "double_launches", "double_launch_word"):
    getattr(D, f).restype = C.c_uint64
D.double_launch_name.restype = C.c_char_p
D.double_unsafe_calls.restype = C.c_int64
for f, a in (("double_capacity", 1), ("double_is_live", 1), ("double_launch_name", 1), ("double_launch_word", 2)):
    getattr(D, f).argtypes = [C.c_uint64] * a
D.double_capture.argtypes = [C.c_uint64, C.c_int]
sys.modules["torch"] = types.SimpleNamespace(_C=None)     # it takes two seconds, and nothing of it is used
from paper_2311_05782_amd import fi
L = fi.lib()
MB, SIDE, OTHER = 1 << 20, 0x5100, 0x5200           # streams are told apart by their handles alone
ANY = 0x10000                                       # operands, faults and records: no kernel runs

def create(M, N, K, device=0):
    h = C.c_void_p()
    st = L.fi_plan_create(C.byref(fi.plan_desc(M, N, K, 16, fi.BF16)), C.c_void_p(ANY), C.c_void_p(ANY), None, C.byref(h))
    assert st == 0, (st, L.fi_last_error())
    return h

def inject(plan, n, stream):
    return L.fi_gemm_inject_batch(plan, C.c_void_p(ANY), C.c_uint32(n), C.c_uint32(1), C.c_void_p(ANY), None, C.c_void_p(stream))

def affected(plan, n, stream):
    return L.fi_gemm_inject_batch_affected(plan, C.c_void_p(ANY), C.c_uint32(n), C.c_uint32(1), C.c_void_p(ANY), C.c_void_p(stream))

def reserve(plan, n, stream):
    return L.fi_plan_reserve(plan, C.c_uint32(n), C.c_void_p(stream))

def names():
    return [D.double_launch_name(i).decode() for i in range(D.double_launches())]

def scratch_of_last_batch():
    at = [i for i, s in enumerate(names()) if "partition_trials" in s][-1]
    return [D.double_launch_word(at, w) for w in range(3)]

def parts_used():
    # the rows' kernel first: the element kernel adds up what it has left
    k = [s for s in names() if "affected_" in s]
    assert len(k) == 2, k
    return "affected_rows" in k[0]
"""


@functools.lru_cache(None)
def _double():
    folder = tempfile.TemporaryDirectory()
    path = os.path.join(folder.name, "hip_runtime_double.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-w", "-I", "/opt/rocm/include",
                    os.path.join(HERE, "hip_runtime_double.cpp"), "-o", path], check=True)
    return folder, path


def run(body):
    code = PRELUDE % dict(root=ROOT, double=_double()[1]) + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], cwd=ROOT, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
