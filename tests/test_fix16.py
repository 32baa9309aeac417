"""The fixed-point coordinates of the int16 lists (eq. (3), Section 3): exact
for every length and slope they are used for, and the bound on the length is
needed (CPU only)."""

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
    out = str(tmp_path_factory.mktemp("fix16") / "fix16_check")
    subprocess.check_call([hipcc, "-O2", "-std=c++17", "-ffp-contract=off",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2009_09500_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "cpp", "fix16_check.cpp")])
    return out


def test_every_length(driver):
    r = subprocess.run([driver], capture_output=True, text=True)
    words = r.stdout.split()
    assert int(words[1]) > 5_000_000 and r.returncode == 0 and int(words[3]) == 0, r.stdout


def test_longer_runs_and_segments_are_caught(driver):
    for args in (["3900", "40"], ["20000", "7"]):
        r = subprocess.run([driver] + args, capture_output=True, text=True)
        assert r.returncode == 1 and int(r.stdout.split()[3]) > 0, (args, r.stdout)
