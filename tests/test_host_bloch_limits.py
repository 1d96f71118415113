"""CPU test of the image-summed list's size limits (no GPU, no kernel):
tests/host/bloch_limits.cpp is compiled with g++ against the library's host
builder and run."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_08935_amd", "csrc")


def test_limits_are_counted_before_the_tables_are_filled(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "bloch_limits")
    subprocess.run([gxx, "-O1", "-g", "-ffp-contract=off", "-std=c++17", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "bloch_limits.cpp"), os.path.join(CSRC, "sphere.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
