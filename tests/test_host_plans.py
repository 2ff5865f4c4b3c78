"""Tiling plans against the workspace they run in (ea_host.cpp), driven over every group size by
tests/native/host_plans_main.cpp.  CPU only."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_every_plan_fits_the_workspace(tmp_path):
    exe = str(tmp_path / "host_plans")
    cmd = ["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(ROOT, "tests", "native", "host_plans_main.cpp"),
           os.path.join(ROOT, "paper_2510_00636_amd", "csrc", "ea_host.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "host plans fit" in r.stdout


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_chosen_score_plans_fit_the_workspace(tmp_path):
    exe = str(tmp_path / "score_choice")
    cmd = ["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(ROOT, "tests", "native", "score_choice_main.cpp"),
           os.path.join(ROOT, "paper_2510_00636_amd", "csrc", "ea_host.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
    assert "score plans fit" in r.stdout
