"""Coulomb tensors on the GPU against the oracle: a sphere of one point, every
shell (one and two density tiles), several sites in one call, spheres over the
cell faces, and planes of the kernel past the work-group's LDS."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402
from oracle import coulomb as C  # noqa: E402
from oracle.orbitals import Site, System, build_sphere  # noqa: E402
from tests.helpers import normwise  # noqa: E402

CASES = {
    "shells": ([8.0, 8.5, 9.0], [27, 28, 31], [(0.3, 8.2, 3.3, 0, 1.6, 2.9), (3.1, 3.0, 0.5, 1, 1.3, 3.4),
                                               (4.2, 0.1, 8.8, 2, 2.0, 3.9), (2.0, 6.0, 5.0, 3, 2.4, 4.1)]),
    "one point": ([4.0, 4.0, 4.0], [8, 8, 8], [(1.0, 1.0, 1.0, 0, 1.0, 0.05)]),
    "own images": ([5.0, 5.0, 5.0], [13, 13, 13], [(0.1, 0.2, 4.9, 2, 1.4, 4.6)]),
    "planes filling LDS": ([6.0, 5.0, 5.0], [8, 93, 93], [(3.1, 2.51, 2.47, 0, 1.3, 2.4)]),
    "planes past LDS": ([6.0, 5.0, 5.0], [12, 100, 100], [(3.1, 2.51, 2.47, 1, 1.3, 2.4), (0.2, 0.3, 1.0, 2, 2.0, 1.0)]),
}


@pytest.mark.parametrize("name", list(CASES))
def test_tensors_match_the_oracle(name):
    cell, ngrid, sites = CASES[name]
    sites = [dict(R=s[:3], l=s[3], zeta=s[4], rc=s[5], species=0) for s in sites]
    hub = H.Hubbard(cell, ngrid, sites)
    hub.coulomb(-1)
    whole = [hub.get_coulomb(i).cpu().numpy() for i in range(hub.nsites)]
    osites = [Site(R=np.array(s["R"]), l=s["l"], zeta=s["zeta"], rc=s["rc"]) for s in sites]
    sys_ = System(cell=cell, ngrid=ngrid, sites=osites, kpts=np.zeros((1, 3)), kweights=np.ones(1), spin="unpolarized")
    for i, s in enumerate(osites):
        ref = C.coulomb_tensor(sys_, s, build_sphere(sys_, s), method="fft")
        # positive sums of up to 5e4^2 terms and an FFT of 1e6 points in FP64
        assert normwise(whole[i], ref) < 1e-12
        # a site's tensor has the same bits whichever sites a call computes
        one = hub.coulomb(i).cpu().numpy()
        assert np.array_equal(one, whole[i])
        for p in ((1, 0, 2, 3), (0, 1, 3, 2), (2, 3, 0, 1)):
            assert np.array_equal(one, one.transpose(p))
    hub.close()
