"""The record of the LDS limits that have been raised (per kernel and device), compiled for the host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1211_5590_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_a_limit_is_recorded_per_kernel_and_device(tmp_path):
    exe = str(tmp_path / "lds_limit")
    built = subprocess.run(["g++", "-std=c++17", "-O1", "-pthread", "-I", CSRC, "-o", exe, os.path.join(HERE, "lds_limit_main.cpp")],
                           capture_output=True, text=True)
    assert built.returncode == 0, built.stderr
    run = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert run.returncode == 0 and run.stdout.strip().endswith("ok"), run.stdout + run.stderr


def test_no_source_keeps_a_limit_of_its_own():
    """Every launcher asks the record: a flag beside a launch would be one for all devices."""
    for name in sorted(os.listdir(CSRC)):
        if name.endswith((".hip", ".hpp")) and name != "lds_limit.hip":
            assert "hipFuncSetAttribute" not in open(os.path.join(CSRC, name)).read(), name
