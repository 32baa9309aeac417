"""How small bit-volume calls deal the volume's words to workgroups when the
segments are not spread over it (CPU only)."""

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
    out = str(tmp_path_factory.mktemp("slabcut") / "slab_cut_check")
    subprocess.check_call([hipcc, "--offload-arch=gfx950", "-O2", "-std=c++17",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2009_09500_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "cpp", "slab_cut_check.cpp")])
    return out


def test_every_cut_covers_and_fits(driver):
    r = subprocess.run([driver], capture_output=True, text=True)
    words = r.stdout.split()
    assert int(words[1]) > 1000 and int(words[3]) > 1000, r.stdout
    assert r.returncode == 0 and int(words[5]) == 0, r.stdout


def test_too_long_runs_are_caught(driver):
    r = subprocess.run([driver, "light"], capture_output=True, text=True)
    assert r.returncode == 1 and int(r.stdout.split()[5]) > 0, r.stdout
