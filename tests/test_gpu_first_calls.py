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
