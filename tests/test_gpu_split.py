"""Chunks shared by several work-groups (launches too small for the chip):
projections, V_U psi and forces against the oracle for chunk lengths from one
entry batch to a whole sphere, one to many columns, both work lists, and a
context whose states sets are projected one at a time (same bits)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402
from oracle import forces as OF  # noqa: E402
from oracle import potential as OV  # noqa: E402
from oracle import projection as OP  # noqa: E402
from oracle.orbitals import Site, System  # noqa: E402
from tests.helpers import normwise  # noqa: E402

CELL, NGRID = (6.0, 6.5, 7.0), (17, 18, 21)
SHELLS = [((0.3, 6.2, 3.3), 2, 2.9), ((3.1, 3.0, 0.5), 3, 2.1), ((5.0, 5.0, 5.0), 0, 0.9), ((1.0, 4.0, 6.0), 1, 3.2)]


@pytest.mark.parametrize("grouped", [True, False])
@pytest.mark.parametrize("states", [1, 6, 70])
@pytest.mark.parametrize("chunk", [64, 100, 512, 8192])
def test_split_chunks_match_the_oracle(chunk, states, grouped):
    sites = [dict(R=R, l=l, zeta=1.7, rc=rc, species=i) for i, (R, l, rc) in enumerate(SHELLS)]
    kpts = np.array([[0.1, -0.2, 0.3], [0.0, 0.25, -0.4]])
    hub = H.Hubbard(CELL, NGRID, sites, kpts=kpts, kweights=[0.4, 0.6], spin="collinear", is_complex=True,
                    precision="f64", chunk=chunk)
    hub.set_worklist(grouped)
    rng = np.random.default_rng(chunk + states)
    psi = rng.normal(size=(4, hub.G, states)) + 1j * rng.normal(size=(4, hub.G, states))
    f = rng.uniform(size=(4, states))
    psi_d, f_d = torch.from_numpy(psi).cuda(), torch.from_numpy(f).cuda()
    c = hub.project(psi_d)
    for q in range(4):
        assert torch.equal(hub.project(psi_d[q:q + 1], sets=(q, 1))[0], c[q])
    n, _, _ = hub.occupations(c, f_d, with_pbar=False, nbar=False)
    ueff = [0.3, -0.2, 0.5, 0.1]
    ue = torch.tensor(ueff, dtype=torch.float64, device="cuda")
    h = torch.from_numpy(psi).cuda()
    hub.apply(ue, n, c, h, alpha=0.8)
    F = hub.forces(psi_d, c, f_d, ue, n)
    osites = [Site(R=np.array(R), l=l, zeta=1.7, rc=rc, species=i) for i, (R, l, rc) in enumerate(SHELLS)]
    sys_ = System(cell=np.array(CELL), ngrid=np.array(NGRID), sites=osites, kpts=kpts, kweights=np.array([0.4, 0.6]),
                  spin="collinear")
    sps = OP.all_spheres(sys_)
    c_ref = OP.project_sphere(sys_, psi, sps)
    # FP64 sums of at most 4000 terms
    assert normwise(c.cpu().numpy(), c_ref) < 1e-13
    nn = n.cpu().numpy()
    V = [OV.potential_matrix(sys_, u, nn[i][:, :s.L, :s.L]) for i, (s, u) in enumerate(zip(osites, ueff))]
    assert normwise(h.cpu().numpy(), psi + 0.8 * OV.apply_fullgrid(sys_, c_ref, V, sps)) < 1e-12
    F_ref = OF.forces_analytic(sys_, c_ref, OF.gradient_projections(sys_, psi, sps), V, f)
    assert normwise(F.cpu().numpy(), F_ref) < 1e-11
    hub.close()
