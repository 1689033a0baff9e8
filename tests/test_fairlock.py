"""The lock that solves resident on the chip share (csrc/fairlock.h): first come,
first served, and one at a time (host code, no GPU needed)."""
import os
import subprocess

import pytest

from paper_1007_3432_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_fair_lock_serves_in_order(tmp_path):
    exe = str(tmp_path / "fairlock_check")
    cmd = ["g++", "-O2", "-std=c++17", "-pthread", "-I", build.CSRC,
           os.path.join(HERE, "native", "fairlock_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        pytest.fail("g++ failed:\n" + r.stderr[-2000:])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
    assert out.stdout.startswith("ok"), out.stdout
