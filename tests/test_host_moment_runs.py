"""CPU test of the moment projection's runs (no GPU, no kernel), which the host
builder marks so that a step allocates no host memory for them:
tests/host/moment_runs.cpp is compiled with g++ against the builder and run."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_08935_amd", "csrc")


def test_every_run_is_marked(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "moment_runs")
    subprocess.run([gxx, "-O1", "-g", "-ffp-contract=off", "-std=c++17", "-fsanitize=address,undefined",
                    "-fno-sanitize-recover=all", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    os.path.join(ROOT, "tests", "host", "moment_runs.cpp"), os.path.join(CSRC, "sphere.cpp"),
                    "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
