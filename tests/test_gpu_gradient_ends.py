"""Rows that the energy gradient clears and writes, for every start and length
of a row relative to 16 and 128 bytes: uncovered rows are zero to their last
column, covered ones are scale 2 g_s dV w f V_U psi (formed here from the sphere
tables), and nothing before, between or behind the rows is written."""

import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402


@pytest.fixture(scope="module", params=["f32", "f64"])
def hub(request):
    hub = H.Hubbard((8.0,) * 3, (10, 11, 12), [dict(R=(4.0, 4.2, 3.9), l=1, zeta=1.5, rc=2.6, species=0)],
                    spin="unpolarized", is_complex=False, precision=request.param)
    yield hub
    hub.close()


@pytest.mark.parametrize("start", [0, 1, 2, 3])
@pytest.mark.parametrize("pad", [0, 1, 5])
@pytest.mark.parametrize("states", [1, 2, 3, 4, 5, 7, 16, 31, 63, 64, 65, 127, 129, 143, 160])
def test_rows_end_where_they_end(hub, states, pad, start):
    S, ld, G = states, states + pad, hub.G
    gen = torch.Generator(device="cuda").manual_seed(1000 * S + 10 * pad + start)
    c = torch.randn((1, hub.J, S), generator=gen, device="cuda", dtype=torch.float64)
    f = torch.rand((1, S), generator=gen, device="cuda", dtype=torch.float64)
    ueff = torch.full((1,), 0.3, dtype=torch.float64, device="cuda")
    n = torch.zeros_like(hub.empty_n())                            # V = U / 2
    store = torch.full((start + G * ld + 8,), 7.0, device="cuda", dtype=hub.state_dtype)
    rows = store[start:start + G * ld]
    hub._stream()
    H._check(H.lib().hub_energy_gradient(hub._ctx, None, 0, S, H._dptr(c), H._dptr(f), H._dptr(ueff), H._dptr(n), 0.7,
                                         rows.data_ptr(), ld, None), "hub_energy_gradient")
    g, _, phi, _ = hub.site_points(0)
    g, phi = torch.from_numpy(g).long().cuda(), torch.from_numpy(phi).cuda()
    want = torch.zeros((G, S), device="cuda", dtype=torch.float64)
    want.index_add_(0, g, phi @ (0.15 * c[0] * (0.7 * 4.0 * hub.dV) * f))
    got = rows.view(G, ld)
    assert torch.all(store[:start] == 7.0) and torch.all(store[start + G * ld:] == 7.0)
    assert torch.all(got[:, S:] == 7.0)
    covered = torch.zeros(G, dtype=torch.bool, device="cuda")
    covered[g] = True
    assert torch.count_nonzero(got[~covered, :S]) == 0
    # one rounding to the storage type of a sum of three products
    bar = 1.2e-7 if hub.precision == "f32" else 1e-15
    assert (got[:, :S].double() - want).abs().max() <= bar * want.abs().max()
