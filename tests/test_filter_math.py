"""The filter's elementary functions, compiled for the host, against 80-bit
values.  Bounds: the last rounding, half a unit, and what the steps before it
leave: the logarithm's series beyond r, below 2^-15, rounded a few times,
against units of 2^-60 up; the exponential's series beyond 1 + r + r^2 / 2,
below 2^-7, rounded a few times, and the terms left out, below 2^-57, against
units of 2^-53.  (The device library's own functions reach 0.63 and 0.86.)"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not installed")
def test_errors(tmp_path):
    exe = str(tmp_path / "filter_math")
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I",
                    os.path.join(ROOT, "paper_1301_4019_amd", "csrc"),
                    os.path.join(ROOT, "tests", "filter_math_main.cpp"), "-o", exe, "-lm"],
                   check=True, capture_output=True, text=True)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stdout
    log_max, cos_max, exp_max = map(float, res.stdout.split())
    assert log_max <= 0.5 + 2.0 ** -5
    assert exp_max <= 0.5 + 2.0 ** -3
    assert cos_max <= 2.0  # of 2^-53
