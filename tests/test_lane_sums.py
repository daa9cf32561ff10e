"""The lanes that store the sums of the wave-wide halving exchange (the
Householder reduction's dot products): each of 1 to 16 sums has exactly one
owner, whatever padding the odd counts bring in."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2609_36692_amd", "csrc")


def test_every_sum_has_one_owner(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "lane_sum_check")
    r = subprocess.run([cxx, "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "lane_sum_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 failure(s)" in r.stdout, r.stdout
