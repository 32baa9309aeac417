"""The fixed-point coordinates of the int16 lists for every slope of some lengths,
the longest among them (CPU only)."""

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
    out = str(tmp_path_factory.mktemp("fix16s") / "fix16_slopes_check")
    subprocess.check_call([hipcc, "-O2", "-std=c++17", "-ffp-contract=off",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2009_09500_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "cpp", "fix16_slopes_check.cpp")])
    return out


@pytest.mark.parametrize("lengths", [range(1, 130), (255, 256, 257, 999, 1024), (2047,), (2048,), (3583,), (3889,), (3899,),
                                     (3900,)])
def test_every_slope(driver, lengths):
    r = subprocess.run([driver] + [str(n) for n in lengths], capture_output=True, text=True)
    words = r.stdout.split()
    assert int(words[1]) > 1_000_000 and r.returncode == 0 and int(words[3]) == 0, r.stdout


def test_too_long_segments_are_caught(driver):
    r = subprocess.run([driver, "4999"], capture_output=True, text=True)
    assert r.returncode == 1, r.stdout
