"""csrc/fastdiv.h, which the kernels use to split a pixel index into image, row and column, against the processor's division
(tests/fastdiv_check.cpp, host code)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_division_by_multiplication_is_exact_for_32_bits(tmp_path):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    exe = str(tmp_path / "fastdiv_check")
    r = subprocess.run([cxx, "-std=c++17", "-O1", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                        "-I", os.path.join(ROOT, "paper_2105_00619_amd", "csrc"),
                        os.path.join(ROOT, "tests", "fastdiv_check.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr
