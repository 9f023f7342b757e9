"""What a context does after an allocation failed, on the CPU: the library's
host side over a stand-in for the HIP runtime (tests/emulate/fake_hip.c), in a
process of its own."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2402_11454_amd", "libgsp.so")

RESULTS_BUFFER = """
import ctypes, sys
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
vp, i64 = ctypes.c_void_p, ctypes.c_int64
limit = ctypes.c_size_t.in_dll(fake, "fake_pinned_limit")
alive = ctypes.c_int.in_dll(fake, "fake_pinned_alive")
ctx = vp()
assert L.gsp_create(0, None, ctypes.byref(ctx)) == 0
limit.value = 65536
off = (i64 * 3)(0, 1, 2)
col = (ctypes.c_int32 * 2)(1, 0)

def batch(graphs):   # graphs of one edge
    n, nnz = (i64 * graphs)(*[2] * graphs), (i64 * graphs)(*[2] * graphs)
    offs, cols = (vp * graphs)(*[ctypes.addressof(off)] * graphs), (vp * graphs)(*[ctypes.addressof(col)] * graphs)
    return L.gsp_load_batch(ctx, graphs, n, nnz, offs, cols, None)

load = lambda: L.gsp_load_csr(ctx, i64(2), i64(2), off, col, None, 0)
assert batch(3) == 0
held = alive.value
assert batch(5000) == -2            # its results do not fit the pinned buffer, and a larger one fails
assert load() == 0 and batch(3) == 0   # the context goes on with the one it has
limit.value = 1 << 30
assert batch(5000) == 0 and load() == 0
assert alive.value == held          # a larger buffer replaces the smaller one
assert L.gsp_destroy(ctx) == 0 and alive.value == 0
"""


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not available")
@pytest.mark.skipif(not os.path.exists(LIB), reason="libgsp.so not built")
def test_context_survives_a_failed_results_buffer(tmp_path):
    fake = str(tmp_path / "libfake_hip.so")
    b = subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", fake,
                        os.path.join(ROOT, "tests", "emulate", "fake_hip.c")], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([sys.executable, "-c", RESULTS_BUFFER, fake, LIB], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])
