"""The score plan that a call launches (host only): the form for five heads per pass where it is chosen, and where it is not."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="no host compiler")
def test_serving_plans_fit_and_deal_every_tile(tmp_path):
    exe = str(tmp_path / "serving_plan")
    cmd = ["g++", "-std=c++17", "-O1", "-o", exe, os.path.join(ROOT, "tests", "native", "serving_plan_main.cpp"),
           os.path.join(ROOT, "paper_2510_00636_amd", "csrc", "ea_host.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout + r.stderr
