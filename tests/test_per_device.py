"""Set-up once on every device, from several threads (host logic, CPU)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_threads_and_devices(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "per_device_check"
    subprocess.run([cxx, "-O2", "-std=c++17", "-pthread", "-I" + os.path.join(ROOT, "paper_2605_18389_amd", "csrc"),
                    os.path.join(ROOT, "tests", "per_device_check.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and r.stdout.strip() == "OK", r.stdout + r.stderr
