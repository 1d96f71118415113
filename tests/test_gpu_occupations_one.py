"""n, N-bar and P-bar where one tile of (k-point, state) pairs holds them all
(at most 64) and where it just does not, for one and two channels and spinors,
with and without P-bar and N-bar, shells of every l, and orbitals beyond those
whose N-bar the occupation kernel forms itself; the batched step against the
separate calls on its c (bitwise).

Tolerance: a sum of at most 65 products of four factors in FP64 is off by at
most 70 x 1.1e-16 < 1e-14 of the sum of magnitudes; P-bar's N-bar adds the
same for its orbitals (at most 150): 1e-13 covers all."""

import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402


def _hub(spin, nk, shells, cplx=True, fixed=True):
    sites = [dict(R=(0.7 * i, 0.5 * i, 0.3 * i), l=l, zeta=1.4, rc=1.6, species=sp) for i, (l, sp) in enumerate(shells)]
    kp = [(0.1 * i, -0.2, 0.3 if cplx else 0.0) for i in range(nk)] if cplx else [(0.0, 0.0, 0.0)]
    hub = H.Hubbard((7.0, 7.0, 7.0), (14, 14, 14), sites, kpts=kp, kweights=[1.0 / nk] * nk, spin=spin,
                    is_complex=cplx, precision="f64")
    for i in range(hub.nsites if fixed else 0):
        hub.set_fixed_ueff(i, 0.2)
    return hub


MIX = [(0, 0), (1, 1), (2, 2), (3, 4), (2, 2)]     # species 3 has no site


@pytest.mark.parametrize("spin,nk,S,cplx", [("unpolarized", 1, 1, False), ("unpolarized", 1, 64, True),
                                            ("unpolarized", 5, 13, True), ("collinear", 2, 32, True),
                                            ("collinear", 1, 65, False), ("spinor", 3, 21, True),
                                            ("spinor", 1, 65, True)])
@pytest.mark.parametrize("shells", [MIX, [(3, i % 2) for i in range(19)]], ids=["mixed", "133 orbitals"])
def test_occupations_against_sums(spin, nk, S, cplx, shells):
    hub = _hub(spin, nk, shells, cplx)
    gen = torch.Generator().manual_seed(5)
    J, nq, ncol = hub.J, hub.nsets, hub.ncol(S)
    c = torch.randn((nq, J, ncol, 2), generator=gen, dtype=torch.float64)
    c = torch.view_as_complex(c) if cplx else c[..., 0].contiguous()
    f = torch.rand((nq, S), generator=gen, dtype=torch.float64)
    n, pbar, nbar = (x.cpu() for x in hub.occupations(c.cuda(), f.cuda()))
    n2, none, _ = hub.occupations(c.cuda(), f.cuda(), with_pbar=False, nbar=False)
    n3, pbar3, _ = hub.occupations(c.cuda(), f.cuda(), nbar=False)
    assert none is None and torch.equal(n2.cpu(), n) and torch.equal(n3.cpu(), n) and torch.equal(pbar3.cpu(), pbar)
    nsig = 2 if spin == "spinor" else 1
    nch = 2 if spin == "collinear" else 1
    cc = c.to(torch.complex128).reshape(nq, J, S, nsig)
    nspec = hub.nspecies
    ref_nb = torch.zeros((nq, nspec, S), dtype=torch.float64)
    orb = 0
    for l, sp in shells:
        ref_nb[:, sp] += (cc[:, orb:orb + 2 * l + 1].abs() ** 2).sum(dim=(1, 3))
        orb += 2 * l + 1
    assert ((nbar - ref_nb).abs() <= 1e-13 * ref_nb).all()
    n, pbar = (x.reshape(hub.nsites, -1, 7, 7) for x in (n, pbar))
    orb = 0
    for i, (l, sp) in enumerate(shells):
        L = 2 * l + 1
        x = cc[:, orb:orb + L]
        orb += L
        for ch in range(nch):
            w = f[ch::nch] / nk
            for got, wt in ((n, w), (pbar, w * ref_nb[ch::nch, sp])):
                for s in range(nsig):
                    for t in range(nsig):
                        a, b = x[ch::nch, :, :, s], x[ch::nch, :, :, t]
                        ref = torch.stack([torch.stack([(wt * a[:, m].conj() * b[:, p]).sum() for p in range(L)])
                                           for m in range(L)])
                        mag = torch.stack([torch.stack([(wt * a[:, m].abs() * b[:, p].abs()).sum() for p in range(L)])
                                           for m in range(L)])
                        blk = got[i, 2 * s + t if nsig == 2 else ch]
                        assert ((blk[:L, :L] - ref).abs() <= 1e-13 * mag).all()
                        assert torch.count_nonzero(blk[L:]) == 0 and torch.count_nonzero(blk[:, L:]) == 0


@pytest.mark.parametrize("spin,S", [("unpolarized", 64), ("unpolarized", 65), ("collinear", 64), ("spinor", 33)])
@pytest.mark.parametrize("fixed", [False, True])
def test_step_equals_separate_calls(spin, S, fixed):
    hub = _hub(spin, 1, MIX, fixed=fixed)
    if not fixed:
        hub.coulomb(-1)
    gen = torch.Generator().manual_seed(6)
    psi = torch.view_as_complex(torch.randn((hub.nsets, hub.G, hub.ncol(S), 2), generator=gen,
                                            dtype=torch.float64)).cuda()
    f = torch.rand((hub.nsets, S), generator=gen, dtype=torch.float64).cuda()
    out = hub.step(psi, f, torch.zeros_like(psi), mode="batched")
    n, pbar, nbar = hub.occupations(out["c"], f)
    U, J, Ueff, status = hub.acbn0(n, pbar)
    for k, v in dict(n=n, pbar=pbar, nbar=nbar, U=U, J=J, Ueff=Ueff, status=status).items():
        assert torch.equal(out[k], v), k
