"""Per-device set-up of kernels: every device that a process drives, once each."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_each_device_is_set_up_once(tmp_path):
    cxx = shutil.which("g++") or shutil.which("clang++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    exe = str(tmp_path / "device_once")
    subprocess.run([cxx, "-std=c++17", "-O1", os.path.join(ROOT, "tests", "c", "device_once.cpp"), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout


def test_no_set_up_is_kept_for_one_device_only():
    """No source keeps the result of a kernel's set-up in a plain static, which the first device to
    come would decide for all."""
    csrc = os.path.join(ROOT, "paper_1306_2461_amd", "csrc")
    for name in sorted(os.listdir(csrc)):
        text = open(os.path.join(csrc, name)).read()
        assert "static const hipError_t" not in text, name
