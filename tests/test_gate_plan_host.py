"""The coset programs that hs_evolve runs, walked on the host as the kernel
walks them and compared with exact Pauli rotations in FP64
(tests/c/gate_plan_check.cpp: random Pauli sums, tile sizes, both coset
sizes, fused, one factor per launch and looped), under AddressSanitizer and
UndefinedBehaviorSanitizer.  Host code only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_coset_programs_equal_exact_rotations(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "gate_plan_check")
    csrc = os.path.join(ROOT, "paper_2606_16959_amd", "csrc")
    cmd = [gxx, "-std=c++17", "-O2", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "c", "gate_plan_check.cpp"),
           os.path.join(csrc, "plan.cpp"), os.path.join(csrc, "gate_plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-2000:]
    assert "programs checked" in run.stdout
