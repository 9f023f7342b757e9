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


GROUPS = """
import ctypes, sys
sys.path.insert(0, sys.argv[3])
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
import paper_2402_11454_amd as gsp
L = gsp.lib()
left, alive = (ctypes.c_int.in_dll(fake, "fake_" + k) for k in ("mallocs_left", "device_alive"))
off, col, w = np.array([0, 1, 2]), np.array([1, 0], np.int32), np.array([1.0, 1.0], np.float32)
opt = gsp.default_options(use_graphs=0, **eval(sys.argv[4]))

def after(mallocs):   # a run with so many device allocations left, then one with enough
    c = gsp.Context(0)
    c._check(L.gsp_pruner_set(c._h, np.zeros(4801, np.float32).ctypes.data, 4801, 0), "set")
    c.load(off, col, w)
    before, seen = alive.value, []
    for n in (mallocs, 1 << 30):
        left.value = n
        # -2: no memory; -3: past its allocations (the stand-in sweeps nothing)
        seen.append((L.gsp_run(c._h, 0.01, 10, ctypes.byref(opt)), alive.value - before))
    left.value = 1 << 30
    c.close()
    return seen

(st, all_of_them), _ = after(1 << 30)
assert st == -3 and all_of_them >= int(sys.argv[5]), (st, all_of_them)
for k in range(all_of_them):
    (first, held), (second, then) = after(k)
    assert first == -2 and second == -3, (k, first, second)
    assert then == all_of_them, f"{then} buffers after a failure at {k}, {all_of_them} without"
assert alive.value == 0
"""


def _run(tmp_path, code, *args):
    fake = str(tmp_path / "libfake_hip.so")
    b = subprocess.run(["gcc", "-O1", "-Wall", "-shared", "-fPIC", "-o", fake,
                        os.path.join(ROOT, "tests", "emulate", "fake_hip.c")], capture_output=True, text=True)
    assert b.returncode == 0, b.stderr
    r = subprocess.run([sys.executable, "-c", code, fake, LIB] + list(args), capture_output=True, text=True,
                       timeout=120)
    assert r.returncode == 0, (r.returncode, r.stderr[-2000:])


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not available")
@pytest.mark.skipif(not os.path.exists(LIB), reason="libgsp.so not built")
def test_context_survives_a_failed_results_buffer(tmp_path):
    _run(tmp_path, RESULTS_BUFFER)


@pytest.mark.skipif(shutil.which("gcc") is None, reason="gcc not available")
@pytest.mark.skipif(not os.path.exists(LIB), reason="libgsp.so not built")
@pytest.mark.parametrize("options, buffers", [("dict()", 14), ("dict(leiden=1)", 16),
                                              ("dict(prune_mode=gsp.PRUNE_LEARNED)", 20),
                                              ("dict(vertex_order=gsp.ORDER_DEGREE)", 22)])
def test_buffers_of_a_run_are_had_together(tmp_path, options, buffers):
    """A run's buffers (levels, refinement, gate, degree order) after each
    of their allocations failed once: the next run has them all."""
    _run(tmp_path, GROUPS, ROOT, options, str(buffers))
