"""Chunks shared by several work-groups: no more of them than a list's longest
chunk has entries for, so that a list of short chunks keeps its workspace and
its sums (against sums over the sphere in torch)."""

import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402


@pytest.mark.parametrize("rc,entries", [(2.1, 64), (2.6, 96)])
def test_short_chunks_are_not_split_past_their_entries(rc, entries):
    # one f shell, its chunk shared by at most two groups of four waves of 8 entries
    S, n, most = 16000, 8, 2

    def context():
        return H.Hubbard((8.0,) * 3, (n,) * 3, [dict(R=(4.0, 4.0, 4.0), l=3, zeta=1.5, rc=rc, species=0)],
                         spin="unpolarized", is_complex=False, precision="f64")

    hub, first = context(), context()
    assert hub.query(5) == 1 and hub.query(10) == 7 and (hub.site_npts[0] + 31) // 32 * 32 == entries
    gen = torch.Generator(device="cuda").manual_seed(1)
    psi = torch.randn((1, n ** 3, S), generator=gen, device="cuda", dtype=torch.float64)
    c = hub.empty_c(S)
    # another context's first call loads the kernels, whose code takes memory too
    first.project(psi, out=c)
    hub._stream()
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    hub.project(psi, out=c)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    # 7 partial rows of 16000 values a split, in pages of 2 MB
    assert used <= most * 7 * S * 8 + (2 << 20)
    g, _, phi, _ = hub.site_points(0)
    want = hub.dV * torch.from_numpy(phi).cuda().T @ psi[0][torch.from_numpy(g).long().cuda()]
    assert (c[0] - want).abs().max() < 1e-13 * want.abs().max() * 10
    # the apply's empty parts leave the rest of the chunk's rows to the others
    n_ = torch.zeros_like(hub.empty_n())
    h = torch.zeros_like(psi)
    hub.apply(torch.full((1,), 0.4, dtype=torch.float64, device="cuda"), n_, c, h)
    ref = torch.zeros_like(psi)
    ref[0].index_add_(0, torch.from_numpy(g).long().cuda(), torch.from_numpy(phi).cuda() @ (0.2 * c[0]))
    assert (h - ref).abs().max() < 1e-13 * ref.abs().max() * 10
    hub.close()
    first.close()
