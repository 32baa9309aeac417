"""The fractions that step a piece inside an LDS brick (eq. (3), Section 3):
23-bit remainders and slopes, rounded up, against the integer divisions they
stand for, over the whole range of N the bricks take (CPU only)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    out = str(tmp_path_factory.mktemp("fix23") / "fix23_check")
    subprocess.check_call([hipcc, "-O2", "-std=c++17", "-ffp-contract=off",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2009_09500_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "cpp", "fix23_check.cpp")])
    return out


def test_every_quotient_of_a_piece(driver):
    r = subprocess.run([driver, "256"], capture_output=True, text=True)
    words = r.stdout.split()
    assert int(words[1]) > 100000 and r.returncode == 0 and int(words[3]) == 0, r.stdout


def test_slopes_rounded_down_are_caught(driver):
    r = subprocess.run([driver, "256", "floor"], capture_output=True, text=True)
    assert r.returncode == 1 and int(r.stdout.split()[3]) > 0, r.stdout
