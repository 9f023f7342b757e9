"""Kernels with barriers inside branches, run on the CPU from their own source
(tests/emulate): every thread of a workgroup has to meet the same barriers
whichever wavefront comes last and whatever other workgroups write meanwhile.
A GPU run shows a mistake here only by chance, and then by hanging or by
wrong sums."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2402_11454_amd", "csrc")
EMULATE = os.path.join(ROOT, "tests", "emulate")


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
@pytest.mark.parametrize("case, source", [("TOTALS", "k_move.hip"), ("PLACES", "k_aggregate.hip"), ("HUBS", "k_move.hip")])
def test_barriers_are_met_by_all(tmp_path, case, source):
    with open(os.path.join(CSRC, source)) as f:
        kernels = f.read().split("}  // namespace\n")[0]   # the kernels come first
    assert "<<<" not in kernels
    src = tmp_path / "kernels.h"
    src.write_text(kernels + "}\n}\n")
    exe = str(tmp_path / "barriers")
    cmd = ["g++", "-std=c++17", "-O1", "-ffp-contract=off", "-w", f"-D{case}", f'-DKERNELS="{src}"',
           "-I", EMULATE, "-I", CSRC, "-o", exe, os.path.join(EMULATE, "barriers.cpp")]
    b = subprocess.run(cmd, capture_output=True, text=True)
    assert b.returncode == 0, b.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, (r.returncode, r.stdout[-2000:])
