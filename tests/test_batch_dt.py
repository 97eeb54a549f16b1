"""The dt kernel of the batched step (ctmhd_workgroup.h), compiled as host code
over fibers that stand for the threads of a workgroup and run in every order of
the wavefronts that its barriers allow."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_every_box_reports_its_dt_of_a_stopping_step(tmp_path):
    exe = str(tmp_path / "batch_dt_check")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-I", os.path.join(ROOT, "tests"),
                           "-I", os.path.join(ROOT, "paper_2609_10816_amd", "csrc"),
                           os.path.join(ROOT, "tests", "batch_dt_check.cpp"), "-o", exe])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
