"""dE_U/dpsi* against hub_apply into a cleared buffer, weighted by w_k f: the
grouped list writes covered rows without reading them and clears the others.
Rows of every alignment, padding columns, several passes (points with more
than 16 functions), a field, spinors, every point covered, few covered, and
the per-site list (every row cleared, layers added)."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402

# cell, grid, shells (R, l, rc), spin, complex, precision, states, padding columns, field
CASES = {
    "few covered": ((9.0, 9.0, 9.0), (21, 22, 23), [((4, 4, 4), 2, 1.5)], "unpolarized", False, "f32", 7, 0, False),
    "wide rows": ((9.0, 9.0, 9.0), (18, 18, 20), [((4, 4, 4), 3, 2.5), ((1, 8, 0), 1, 2.0)], "unpolarized", False, "f32",
                  260, 4, False),
    "padded": ((7.0, 7.0, 7.0), (15, 16, 17), [((1, 1, 1), 2, 2.5)], "collinear", True, "f64", 5, 3, False),
    "passes": ((5.0, 5.0, 5.0), (11, 12, 13), [((1, 1, 1), 2, 4.0), ((3, 3, 3), 1, 3.5)], "collinear", True, "f32", 33, 1,
               False),
    "passes, field": ((5.0, 5.0, 5.0), (11, 12, 13), [((1, 1, 1), 2, 4.0), ((3, 3, 3), 1, 3.5)], "collinear", True,
                      "f64", 9, 0, True),
    "spinor": ((6.0, 6.0, 9.0), (13, 13, 20), [((1, 1, 1), 1, 3.0), ((4, 4, 6), 2, 2.0)], "spinor", True, "f32", 12, 0,
               True),
}


@pytest.mark.parametrize("grouped", [True, False])
@pytest.mark.parametrize("name", list(CASES))
def test_gradient_equals_apply_into_zeros(name, grouped):
    cell, ngrid, shells, spin, cplx, prec, S, pad, field = CASES[name]
    sites = [dict(R=R, l=l, zeta=1.5, rc=rc, species=i) for i, (R, l, rc) in enumerate(shells)]
    kp = [(0.1, -0.2, 0.3), (0.0, 0.25, 0.0)] if cplx else [(0.0, 0.0, 0.0)]
    hub = H.Hubbard(cell, ngrid, sites, kpts=kp, kweights=[1.0 / len(kp)] * len(kp), spin=spin, is_complex=cplx,
                    precision=prec)
    hub.set_worklist(grouped)
    if field:
        hub.set_vector_potential([0.1, 0.2, -0.1])
    gen = torch.Generator().manual_seed(3)
    ncol, nq = hub.ncol(S), hub.nsets
    full = torch.randn((nq, hub.G, ncol + pad, 2), generator=gen, dtype=torch.float64)
    psi = (torch.view_as_complex(full) if cplx else full[..., 0].contiguous()).to(hub.state_dtype).cuda()
    f = torch.rand((nq, S), generator=gen, dtype=torch.float64).cuda()
    c = hub.project(psi, nstates=S)
    n, _, _ = hub.occupations(c, f, with_pbar=False, nbar=False)
    ueff = torch.full((hub.nsites,), 0.3, dtype=torch.float64, device="cuda")
    # the buffer holds garbage before the call; the library's own is empty()
    gpsi = torch.full_like(psi, float("nan"))
    H._check(H.lib().hub_energy_gradient(hub._ctx, None, 0, S, H._dptr(c), H._dptr(f), H._dptr(ueff), H._dptr(n), 0.7,
                                         H._dptr(gpsi), psi.stride(1), None), "hub_energy_gradient")
    ref = torch.zeros_like(psi)
    nspin = 2 if spin == "collinear" else 1
    w = torch.tensor(hub.kweights, dtype=torch.float64, device="cuda").repeat_interleave(nspin)[:, None] * f
    gs = 2.0 if spin == "unpolarized" else 1.0
    hub.apply(ueff, n, c, ref, alpha=0.7 * 2.0 * gs * hub.dV, colscale=w.contiguous(), nstates=S)
    torch.cuda.synchronize()
    if pad:
        assert torch.isnan(gpsi[:, :, ncol:]).all()
    a, b = gpsi[:, :, :ncol], ref[:, :, :ncol]
    assert torch.equal(a == 0, b == 0)
    # one rounding to the storage type of sums whose weights differ by rounding
    bar = 4e-7 if prec == "f32" else 1e-14
    assert float((a - b).abs().max() / b.abs().max()) < bar
    hub.close()
