"""CPU test of the Bloch-summed work list (no GPU, no kernel).

tests/host/bloch_tables.cpp is compiled with g++ against the library's host
builder (sphere.cpp), plain and under host AddressSanitizer and
UndefinedBehaviorSanitizer; it checks every index and sums the list against
the states as the projection kernel does.  The sums must equal the oracle's
projections: spheres past half the cell with several images, one and several
passes, chunks of one to sixteen functions, generic k-points."""

import os
import shutil
import struct
import subprocess

import numpy as np
import pytest

from oracle import projection as P
from oracle.orbitals import Site, System
from tests.helpers import normwise

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1711_08935_amd", "csrc")

CASES = [
    # 16 functions in one pass, many images
    ([5.0, 5.5, 6.0], [10, 11, 12], [Site(R=[0.1, 0.2, 5.9], l=2, zeta=1.2, rc=4.9),
                                     Site(R=[2.5, 2.6, 3.0], l=2, zeta=1.4, rc=4.0, species=1),
                                     Site(R=[4.0, 1.0, 1.0], l=1, zeta=1.2, rc=3.0, species=2),
                                     Site(R=[1.0, 4.0, 4.0], l=1, zeta=1.2, rc=3.0, species=2)], [0.25, -0.25, 0.5]),
    # 20 functions: two passes; an s shell that covers few points
    ([4.0, 4.0, 4.0], [9, 8, 10], [Site(R=[0.0, 0.0, 0.0], l=3, zeta=1.2, rc=3.9),
                                   Site(R=[2.0, 2.0, 2.0], l=3, zeta=1.2, rc=3.5, species=1),
                                   Site(R=[1.0, 3.0, 0.5], l=2, zeta=1.5, rc=2.0, species=2),
                                   Site(R=[3.0, 1.0, 2.5], l=0, zeta=1.0, rc=0.7, species=3)], [0.1, 0.37, -0.2]),
]
SANITIZE = ["-g", "-fno-omit-frame-pointer", "-fsanitize=address,undefined", "-fno-sanitize-recover=all"]


@pytest.fixture(scope="module", params=["plain", "sanitized"])
def checker(request, tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("bloch") / "bloch_tables")
    extra = SANITIZE if request.param == "sanitized" else []
    subprocess.run([gxx, "-O2", "-ffp-contract=off", "-std=c++17", *extra, "-I", os.path.join(ROOT, "include"), "-I",
                    CSRC, os.path.join(ROOT, "tests", "host", "bloch_tables.cpp"), os.path.join(CSRC, "sphere.cpp"),
                    "-o", exe], check=True)
    return exe


@pytest.mark.parametrize("case", range(len(CASES)))
def test_bloch_list_sums_to_the_projections(checker, tmp_path, case):
    cell, ngrid, sites, k = CASES[case]
    sys_ = System(cell=cell, ngrid=ngrid, sites=sites, kpts=np.array([k]), kweights=np.ones(1), spin="unpolarized")
    S = 3
    rng = np.random.default_rng(case)
    psi = rng.normal(size=(1, sys_.G, S)) + 1j * rng.normal(size=(1, sys_.G, S))
    inp, out = tmp_path / "in.bin", tmp_path / "out.bin"
    with open(inp, "wb") as f:
        f.write(struct.pack("3d", *cell) + struct.pack("3i", *ngrid) + struct.pack("i", len(sites)))
        for s in sites:
            f.write(struct.pack("3d", *s.R) + struct.pack("i", s.l) + struct.pack("2d", s.zeta, s.rc) +
                    struct.pack("i", s.species))
        f.write(struct.pack("3d", *k) + struct.pack("i", S))
        f.write(np.ascontiguousarray(psi[0]).tobytes())
    r = subprocess.run([checker, str(inp), str(out)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout + r.stderr
    got = np.fromfile(out, dtype=np.complex128).reshape(-1, S)
    # FP64 sums of at most 5000 terms
    assert normwise(got, P.project_sphere(sys_, psi, P.all_spheres(sys_))[0]) < 1e-13
