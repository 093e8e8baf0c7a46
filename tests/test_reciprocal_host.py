"""The kernels' reciprocal and division sequences, compiled for the CPU with
perturbed reciprocal estimates, against the IEEE quotient: equal, whatever the
estimate within the hardware's error (and twice that), also where the quotient
lies as near to the middle of two doubles as a quotient can."""
import os
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2007_01416_amd", "csrc")


@pytest.mark.parametrize("n", [1000000])
def test_correctly_rounded_from_any_estimate(tmp_path, n):
    exe = str(tmp_path / "reciprocal_host")
    cmd = ["g++", "-std=c++20", "-O2", "-ffp-contract=off", "-I", os.path.join(HERE, "host_kernels"), "-I", CSRC,
           os.path.join(HERE, "host_kernels", "reciprocal_host.cpp"), "-o", exe, "-pthread"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe, str(n)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    bad_r, bad_d, hard = map(int, r.stdout.split())
    assert hard > n // 4 and bad_r == 0 and bad_d == 0, r.stdout
