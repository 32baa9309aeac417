"""The 32-bit fractions that step an axis under the Euclidean N of eq. (1): exact for
the lengths they are used for, and the rounding and the bounds are needed (CPU
only)."""

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
    out = str(tmp_path_factory.mktemp("fix32") / "fix32_check")
    subprocess.check_call([hipcc, "-O2", "-std=c++17", "-ffp-contract=off",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2009_09500_amd", "csrc"),
                           "-o", out, os.path.join(ROOT, "tests", "cpp", "fix32_check.cpp")])
    return out


@pytest.mark.parametrize("form,longest", [("walk", 32767), ("list", 32767), ("piece", 16384)])
def test_every_step(driver, form, longest):
    r = subprocess.run([driver, form, str(longest)], capture_output=True, text=True)
    words = r.stdout.split()
    assert int(words[1]) > 8000 and r.returncode == 0 and int(words[3]) == 0, r.stdout


@pytest.mark.parametrize("args", [("walk", "32767", "floor"), ("walk", "65000"), ("list", "32767", "floor"),
                                  ("list", "65000"), ("list", "32767", "unsigned"), ("piece", "16384", "floor"),
                                  ("piece", "16384", "steps"), ("piece", "32767")])
def test_mistakes_are_caught(driver, args):
    r = subprocess.run([driver, *args], capture_output=True, text=True)
    assert r.returncode == 1 and int(r.stdout.split()[3]) > 0, (args, r.stdout)
