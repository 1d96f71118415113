"""hub_coulomb between captured steps: the projection workspace stays where it
is, so the library's step graph is kept (hub_query 16 counts captures) and so is
a graph that the caller captured on it; a context's first Coulomb call leaves
its scratch as that workspace."""

import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402


def _hub():
    hub = H.Hubbard((10.0,) * 3, (32,) * 3, [dict(R=(5.0, 5.0, 5.1), l=3, zeta=1.5, rc=4.0, species=0)],
                    spin="unpolarized", is_complex=False, precision="f64")
    hub.set_fixed_ueff(0, 0.3)
    return hub


def test_captured_steps_keep_their_workspace():
    hub = _hub()
    S = 4
    psi = torch.randn((1, hub.G, S), device="cuda", dtype=torch.float64)
    f = torch.rand((1, S), device="cuda", dtype=torch.float64)
    bufs, h = hub.step_buffers(S), torch.zeros_like(psi)
    hub.step(psi, f, h, mode="graph", bufs=bufs)                   # a workspace of a few kilobytes
    first = bufs["c"].clone()
    assert hub.query(16) == 1
    hub.coulomb(-1)                                                # needs megabytes
    want = hub.get_coulomb(0).clone()
    for _ in range(3):
        bufs["c"].zero_()
        hub.step(psi, f, h, mode="graph", bufs=bufs)
        assert torch.equal(bufs["c"], first)
        assert torch.equal(hub.coulomb(0), want)
    assert hub.query(16) == 1
    hub.close()


def test_first_call_leaves_the_workspace():
    hub = _hub()
    hub.coulomb(-1)
    before = hub.query(15)
    hub.project(torch.randn((1, hub.G, 4), device="cuda", dtype=torch.float64))
    hub.coulomb(-1)
    assert hub.query(15) == before
    hub.close()
