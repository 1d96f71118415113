"""Allocations of a new context's first calls (hub_query 15): the occupations
of one tile of (k-point, state) pairs are summed in one launch that needs no
partial sums in memory, and allocate none; more pairs do."""

import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from tests.test_gpu_occupations_one import MIX, _hub  # noqa: E402


@pytest.mark.parametrize("spin,nk,states,calls,step", [("unpolarized", 1, 64, 0, 0), ("spinor", 3, 21, 0, 0),
                                                       ("collinear", 2, 32, 0, 1), ("collinear", 2, 33, 1, 1)])
def test_occupations_allocate_only_what_they_use(spin, nk, states, calls, step):
    hub = _hub(spin, nk, MIX)
    gen = torch.Generator(device="cuda").manual_seed(states)
    psi = torch.randn((hub.nsets, hub.G, hub.ncol(states)), generator=gen, device="cuda", dtype=hub.state_dtype)
    f = torch.rand((hub.nsets, states), generator=gen, device="cuda", dtype=torch.float64)
    c = hub.project(psi)
    before = hub.query(15)
    n, pbar, nbar = hub.occupations(c, f)
    assert hub.query(15) - before == calls
    h = torch.zeros_like(psi)
    hub.apply(torch.full((hub.nsites,), 0.2, dtype=torch.float64, device="cuda"), n, c, h)
    before = hub.query(15)
    b = hub.step(psi, f, torch.zeros_like(psi), mode="batched")
    # two channels are summed by two launches of the step
    assert hub.query(15) - before == step - calls
    assert torch.equal(b["n"], n) and torch.equal(b["pbar"], pbar) and torch.equal(b["nbar"], nbar)
    hub.close()


@pytest.mark.parametrize("ld,calls", [(40, 0), (4096, 0), (4128, 1)])
def test_apply_allocates_for_long_rows_only(ld, calls):
    # complex rows: the row that padding entries write holds up to 8192 values from hub_finalize on
    hub = _hub("unpolarized", 1, MIX[:2])
    gen = torch.Generator(device="cuda").manual_seed(ld)
    c = torch.randn((1, hub.J, 40), generator=gen, device="cuda", dtype=torch.complex128)
    n, _, _ = hub.occupations(c, torch.ones((1, 40), device="cuda", dtype=torch.float64))
    ueff = torch.full((hub.nsites,), 0.2, dtype=torch.float64, device="cuda")
    out = []
    for width, new in ((ld, calls), (40, 0)):
        h = torch.zeros((1, hub.G, width), device="cuda", dtype=hub.state_dtype)
        before = hub.query(15)
        hub.apply(ueff, n, c, h[:, :, :40])
        assert hub.query(15) - before == new
        out.append(h[:, :, :40].clone())
        assert torch.count_nonzero(h[:, :, 40:]) == 0
    assert torch.equal(*out) and torch.count_nonzero(out[0]) > 0
    hub.close()
