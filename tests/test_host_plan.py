"""How the one-wavefront solve lies in lanes and in LDS (csrc/cost_plan.h), by a small host program,
tests/host/plan_check.cpp: whole numbers, no GPU."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_plan(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = tmp_path / "plan_check"
    build = subprocess.run(
        [cxx, "-std=c++17", "-O1", "-Wall", "-I", os.path.join(ROOT, "paper_2407_14843_amd", "csrc"),
         os.path.join(ROOT, "tests", "host", "plan_check.cpp"), "-o", str(exe)],
        capture_output=True, text=True, timeout=300)
    assert build.returncode == 0, build.stderr[-2000:]
    run = subprocess.run([str(exe)], capture_output=True, text=True, timeout=120)
    assert run.returncode == 0, run.stdout[-2000:]
    assert "plan ok" in run.stdout
