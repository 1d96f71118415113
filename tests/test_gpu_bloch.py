"""Bloch-summed work list (points with more than 16 (orbital, image) functions,
complex states) against the oracle: one and two passes, chunks of up to 8 and
up to 16 functions, column counts around the kernels' 16- and 32-column tiles,
both precisions, spinors, ranges of state sets (same bits), and the grouped
list's passes, which a field takes."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402
from oracle import potential as OV  # noqa: E402
from oracle import projection as OP  # noqa: E402
from oracle.orbitals import Site, System  # noqa: E402
from tests.helpers import normwise  # noqa: E402

SYSTEMS = {
    # 16 functions in one pass
    "one pass": ((5.0, 5.5, 6.0), (13, 14, 15), [((0.1, 0.2, 5.9), 2, 4.9), ((2.5, 2.6, 3.0), 2, 4.0),
                                                 ((4.0, 1.0, 1.0), 1, 3.0), ((1.0, 4.0, 4.0), 1, 3.0)]),
    # 20 functions in two passes, the s shell on few points
    "two passes": ((4.0, 4.0, 4.0), (13, 12, 15), [((0.0, 0.0, 0.0), 3, 3.9), ((2.0, 2.0, 2.0), 3, 3.5),
                                                   ((1.0, 3.0, 0.5), 2, 2.0), ((3.0, 1.0, 2.5), 0, 0.7)]),
    # at most 6 functions, seen through many images
    "few functions": ((3.0, 3.0, 3.5), (9, 10, 11), [((0.2, 0.1, 0.0), 1, 4.0), ((1.5, 1.5, 1.5), 1, 2.5)]),
}


@pytest.mark.parametrize("prec", ["f32", "f64"])
@pytest.mark.parametrize("spin,states", [("collinear", 1), ("collinear", 16), ("collinear", 17), ("collinear", 33),
                                         ("spinor", 8), ("spinor", 20), ("unpolarized", 70)])
@pytest.mark.parametrize("name", list(SYSTEMS))
def test_projections_and_potential(name, spin, states, prec):
    cell, ngrid, shells = SYSTEMS[name]
    sites = [dict(R=R, l=l, zeta=1.3, rc=rc, species=i) for i, (R, l, rc) in enumerate(shells)]
    kpts = np.array([[0.1, -0.2, 0.3], [0.0, 0.25, -0.4]])
    hub = H.Hubbard(cell, ngrid, sites, kpts=kpts, kweights=[0.4, 0.6], spin=spin, is_complex=True, precision=prec)
    assert hub.query(14) > 1                                       # the grouped list needs passes
    ncol, nq = hub.ncol(states), hub.nsets
    rng = np.random.default_rng(states)
    raw = rng.normal(size=(nq, hub.G, ncol)) + 1j * rng.normal(size=(nq, hub.G, ncol))
    psi = torch.from_numpy(raw).to(hub.state_dtype).cuda()
    used = psi.cpu().numpy().astype(np.complex128)
    f = torch.from_numpy(rng.uniform(size=(nq, states))).cuda()
    c = hub.project(psi)
    for q in range(nq):
        assert torch.equal(hub.project(psi[q:q + 1], sets=(q, 1))[0], c[q])
    n, _, _ = hub.occupations(c, f, with_pbar=False, nbar=False)
    ueff = [0.3, -0.2, 0.5, 0.1][:hub.nsites]
    ue = torch.tensor(ueff, dtype=torch.float64, device="cuda")
    h = psi.clone()
    hub.apply(ue, n, c, h, alpha=0.8)
    part = psi[1:2].clone()
    hub.apply(ue, n, c[1:2].contiguous(), part, alpha=0.8, sets=(1, 1))
    assert torch.equal(part[0], h[1])
    osites = [Site(R=np.array(R), l=l, zeta=1.3, rc=rc, species=i) for i, (R, l, rc) in enumerate(shells)]
    sys_ = System(cell=np.array(cell), ngrid=np.array(ngrid), sites=osites, kpts=kpts, kweights=np.array([0.4, 0.6]),
                  spin=spin)
    sps = OP.all_spheres(sys_)
    wide = used.reshape(nq, hub.G, states, 2) if spin == "spinor" else used
    c_ref = OP.project_sphere(sys_, wide, sps)
    # FP64 sums of at most 2e4 terms of random sign
    assert normwise(c.cpu().numpy().reshape(c_ref.shape), c_ref) < 1e-12
    nn = n.cpu().numpy()
    blocks = [nn[i][:, :s.L, :s.L] for i, s in enumerate(osites)]
    if spin == "spinor":
        blocks = [b.reshape(2, 2, b.shape[1], b.shape[2]) for b in blocks]
    V = [OV.potential_matrix(sys_, u, b) for u, b in zip(ueff, blocks)]
    h_ref = wide + 0.8 * OV.apply_fullgrid(sys_, c_ref, V, sps)
    assert normwise(h.cpu().numpy().reshape(h_ref.shape), h_ref) < (1e-12 if prec == "f64" else 1.2e-7)
    # under a vanishing field the passes of the grouped list give the same sums
    # (in FP32 storage they round the row once per pass, so FP64 only)
    hub.set_vector_potential([0.0, 0.0, 0.0])
    assert normwise(hub.project(psi).cpu().numpy(), c.cpu().numpy()) < 1e-13
    if prec == "f64":
        h2 = psi.clone()
        hub.apply(ue, n, c, h2, alpha=0.8)
        assert normwise(h2.cpu().numpy(), h.cpu().numpy()) < 1e-13
    hub.close()
