"""The projection workspace of a context that has seen a number of states does
not grow for fewer (small launches share their chunks among more work-groups,
each with partial rows of its own): a graph that a caller captured on it, or a
capture in progress, would lose it."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402
from tests.test_gpu_bloch_route import _context  # noqa: E402


def _shells(spin, cplx, prec):
    sites = [dict(R=(4.0 + 2.0 * i, 4.0, 4.0), l=2 - i, zeta=1.5, rc=3.0, species=i) for i in range(2)]
    hub = H.Hubbard((10.0,) * 3, (20,) * 3, sites, spin=spin, is_complex=cplx, precision=prec)
    for i in range(2):
        hub.set_fixed_ueff(i, 0.3)
    return hub


@pytest.mark.parametrize("make", [
    lambda: _shells("unpolarized", False, "f32"), lambda: _shells("collinear", True, "f64"),
    lambda: _context("two passes", rc=0.9), lambda: _context("few functions", spin="spinor")],
    ids=["real", "complex", "image-summed", "image-summed spinors"])
def test_fewer_states_find_the_workspace(make):
    most = 700
    hub = make()
    psi = torch.randn((hub.nsets, hub.G, hub.ncol(most)), device="cuda", dtype=hub.state_dtype)
    f = torch.rand((hub.nsets, most), device="cuda", dtype=torch.float64)
    c = hub.project(psi)
    n, _, _ = hub.occupations(c, f)
    ueff = torch.full((hub.nsites,), 0.2, dtype=torch.float64, device="cuda")
    hub.forces(psi, c, f, ueff, n)
    hub.forces(psi, c, f, ueff, n, form="state")
    seen = hub.query(15)
    for S in sorted({*range(1, 40), *np.unique(np.geomspace(40, most, 60).astype(int)).tolist()}):
        part = hub.project(psi, nstates=S)
        assert hub.query(15) == seen, S
        hub.forces(psi, part, f[:, :S].contiguous(), ueff, n, nstates=S)
        hub.forces(psi, part, f[:, :S].contiguous(), ueff, n, nstates=S, form="state")
        assert hub.query(15) == seen, S
    hub.close()
