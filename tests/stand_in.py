"""Runs a piece of a test in a process of its own where libtid calls the
stand-in HIP runtime (stand_in_hip.c) instead of the real one."""
import json
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))

PRELUDE = r"""
import ctypes, json, sys
hip = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)    # before libtid: its calls go here
sys.path.insert(0, sys.argv[2])
from paper_1807_01409_amd import _lib as L
lib = L.load_library()
def word(name, kind=ctypes.c_uint64):
    return kind.in_dll(hip, name)
def kernels():
    text = (ctypes.c_char * (1 << 20)).in_dll(hip, "launched").value.decode()
    return [k for k in text.split("\n") if k]
def context():
    ctx = ctypes.c_void_p()
    assert lib.tid_ctx_create(0, None, L.ALLOC_FN(), L.FREE_FN(), None, ctypes.byref(ctx)) == 0
    return ctx
def device(nbytes):
    p = ctypes.c_void_p()
    assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(nbytes)) == 0
    return p
def table(ctx, nrows, ncols=1, first=0):
    col = device(4 * max(nrows, 1))
    cols = (ctypes.c_void_p * ncols)(*[col.value] * ncols)
    names = (ctypes.c_int32 * ncols)(*range(first, first + ncols))
    t = ctypes.c_void_p()
    st = lib.tid_table_from_columns(ctx, cols, ncols, names, nrows, 1, ctypes.byref(t))
    assert st == 0, st
    return t
def error(ctx):
    return lib.tid_last_error(ctx).decode()
out = {}
"""


def run(tmp_path, code, timeout=120):
    """`code` after PRELUDE, in its own process; what it left in `out`."""
    so = str(tmp_path / "stand_in_hip.so")
    subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", so,
                    os.path.join(HERE, "stand_in_hip.c")], check=True)
    # freed host memory is overwritten, and never unmapped
    env = dict(os.environ, MALLOC_PERTURB_="165", MALLOC_MMAP_THRESHOLD_=str(1 << 30),
               MALLOC_TRIM_THRESHOLD_=str(1 << 40))
    r = subprocess.run([sys.executable, "-c", PRELUDE + code + "\nprint(json.dumps(out))", so,
                        os.path.dirname(HERE)], capture_output=True, text=True, env=env,
                       timeout=timeout)
    assert r.returncode == 0, r.stderr[-2000:]
    return json.loads(r.stdout.splitlines()[-1])
