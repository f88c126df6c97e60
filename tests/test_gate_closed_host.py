"""The closure check of the coset programs can fail: entries planted outside
a factor's cosets are found (tests/c/gate_closed_check.cpp).  Host code only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_entries_outside_the_cosets_are_found(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "gate_closed_check")
    csrc = os.path.join(ROOT, "paper_2606_16959_amd", "csrc")
    cmd = [gxx, "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), os.path.join(ROOT, "tests", "c", "gate_closed_check.cpp"),
           os.path.join(csrc, "plan.cpp"), os.path.join(csrc, "gate_plan.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-2000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0, run.stdout[-2000:] + run.stderr[-2000:]
    assert "planted entries checked" in run.stdout
