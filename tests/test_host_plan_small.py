"""Small batches in the attend planner (host C++, no GPU): compiles the planner together with a checker and runs it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2605_26289_amd", "csrc")


def test_small_batches_cover_every_row_and_key_once(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "plan_small_check")
    cmd = [cxx, "-std=c++17", "-O1", "-g", "-pthread", os.path.join(ROOT, "tests", "plan_small_check.cpp"),
           os.path.join(CSRC, "plan.cpp"), os.path.join(CSRC, "pool.cpp"), "-o", exe]
    built = subprocess.run(cmd, capture_output=True, text=True)
    assert built.returncode == 0, built.stderr[-3000:]
    run = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert run.returncode == 0 and "failures 0" in run.stdout, (run.stdout[-3000:], run.stderr[-2000:])
