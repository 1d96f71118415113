"""CPU test of the Coulomb tensors' work list (no GPU, no kernel).

tests/host/coulomb_plan.cpp is compiled with g++ against the library's host
builder (sphere.cpp), plain and under host AddressSanitizer and
UndefinedBehaviorSanitizer; it checks every index and sums the work items in
plain loops.  The tensors must equal the oracle's direct double sum: every
shell, spheres that wrap over the cell faces and reach their own images, a
sphere of one point, uneven grids."""

import os
import shutil
import struct
import subprocess

import numpy as np
import pytest

from oracle import coulomb as C
from oracle.orbitals import Site, System, build_sphere
from tests.helpers import normwise

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_08935_amd", "csrc")

CASES = [
    ([6.0, 6.5, 7.0], [15, 16, 18], [Site(R=[0.3, 6.2, 3.3], l=2, zeta=1.6, rc=2.4),
                                     Site(R=[3.1, 3.0, 0.5], l=1, zeta=1.3, rc=1.9, species=1)]),
    ([3.0, 5.0, 4.0], [8, 11, 10], [Site(R=[0.0, 0.0, 0.0], l=3, zeta=1.2, rc=2.6),
                                    Site(R=[1.5, 4.99, 0.01], l=0, zeta=1.0, rc=1.3, species=1)]),
    # one point; a sphere thin along x with long lines
    ([4.0, 4.0, 4.0], [8, 8, 40], [Site(R=[1.0, 1.0, 1.0], l=0, zeta=1.0, rc=0.05),
                                   Site(R=[2.2, 2.1, 2.05], l=1, zeta=1.0, rc=1.2, species=1)]),
]
SANITIZE = ["-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]


@pytest.fixture(scope="module", params=["plain", "sanitized"])
def checker(request, tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("coulomb") / "coulomb_plan")
    extra = SANITIZE if request.param == "sanitized" else []
    subprocess.run([gxx, "-O2", "-ffp-contract=off", "-std=c++17", *extra, "-I", os.path.join(ROOT, "include"), "-I",
                    CSRC, os.path.join(ROOT, "tests", "host", "coulomb_plan.cpp"), os.path.join(CSRC, "sphere.cpp"),
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("case", range(len(CASES)))
def test_items_sum_to_the_direct_tensor(checker, tmp_path, case):
    cell, ngrid, sites = CASES[case]
    inp, out = tmp_path / "in.bin", tmp_path / "out.bin"
    with open(inp, "wb") as f:
        f.write(struct.pack("3d", *cell) + struct.pack("3i", *ngrid) + struct.pack("i", len(sites)))
        for s in sites:
            f.write(struct.pack("3d", *s.R) + struct.pack("i", s.l) + struct.pack("2d", s.zeta, s.rc) +
                    struct.pack("i", s.species))
    r = subprocess.run([checker, str(inp), str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    got = np.fromfile(out)
    sys_ = System(cell=cell, ngrid=ngrid, sites=sites, kpts=np.zeros((1, 3)), kweights=np.ones(1), spin="unpolarized")
    o = 0
    for s in sites:
        ref = C.coulomb_tensor(sys_, s, build_sphere(sys_, s), method="direct")
        t = got[o:o + s.L ** 4].reshape((s.L,) * 4)
        o += s.L ** 4
        # sums of at most 1500^2 terms: rounding far below 1e-12 of the largest entry
        assert normwise(t, ref) < 1e-12
    assert o == got.size
