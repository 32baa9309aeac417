"""The host slots of calls that ask for a total (CPU only)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_slots_come_back(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "slots_check")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-pthread", "-I", os.path.join(ROOT, "paper_2009_09500_amd", "csrc"),
                           "-o", exe, os.path.join(ROOT, "tests", "cpp", "slots_check.cpp")])
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout
