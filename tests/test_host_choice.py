"""Tile and launch choices of the host logic (bf_host.cpp, no HIP) whose lines
were drawn by measurement: tests/host_choice_check.cpp, built with g++."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1412_4907_amd", "csrc")


@pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")
def test_host_choices(tmp_path):
    exe = str(tmp_path / "host_choice_check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, "-I", os.path.join(ROOT, "include"),
                        os.path.join(CSRC, "bf_host.cpp"),
                        os.path.join(ROOT, "tests", "host_choice_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.startswith("OK"), r.stdout + r.stderr
