"""Which work list the calls take (hub_query 17: image-summed list built, 18:
projections and applies that took it), so that tests of that list's results
cannot pass on the grouped list's passes; and that an apply over it uses
nothing that a second apply on another stream would overwrite."""

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402
from tests.test_gpu_bloch import SYSTEMS  # noqa: E402

KPTS = [[0.1, -0.2, 0.3], [0.0, 0.25, -0.4]]


def _context(name="two passes", spin="collinear", prec="f64", rc=1.0, **kw):
    cell, ngrid, shells = SYSTEMS[name]
    sites = [dict(R=R, l=l, zeta=1.3, rc=r * rc, species=i) for i, (R, l, r) in enumerate(shells)]
    kw.setdefault("is_complex", True)
    if kw["is_complex"]:
        kw.update(kpts=np.array(KPTS), kweights=[0.4, 0.6])
    hub = H.Hubbard(cell, ngrid, sites, spin=spin, precision=prec, **kw)
    for i in range(hub.nsites):
        hub.set_fixed_ueff(i, 0.3 - 0.2 * i)
    return hub


def _inputs(hub, states, seed=0):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    psi = torch.randn((hub.nsets, hub.G, hub.ncol(states)), generator=gen, device="cuda", dtype=hub.state_dtype)
    f = torch.rand((hub.nsets, states), generator=gen, device="cuda", dtype=torch.float64)
    return psi, f


@pytest.mark.parametrize("name", list(SYSTEMS))
def test_calls_take_the_list(name):
    hub = _context(name)
    assert hub.query(14) > 1 and hub.query(17) == 1
    psi, f = _inputs(hub, 48)
    bufs = hub.step_buffers(48)

    def used(call):
        before = hub.query(18)
        call()
        return hub.query(18) - before

    def step(mode):
        return lambda: hub.step(psi, f, torch.zeros_like(psi), mode=mode, bufs=bufs)

    c, h = hub.project(psi), torch.zeros_like(psi)
    n, _, _ = hub.occupations(c, f)
    ueff = torch.full((hub.nsites,), 0.2, dtype=torch.float64, device="cuda")
    calls = [lambda: hub.project(psi), lambda: hub.project(psi[1:2], sets=(1, 1)), lambda: hub.apply(ueff, n, c, h)]
    assert [used(x) for x in calls] == [1, 1, 1]
    assert used(step("batched")) == 2 and used(step("persite")) == 0
    hp = torch.zeros_like(psi)
    graph = lambda: hub.step(psi, f, hp, mode="graph", bufs=bufs)  # noqa: E731
    assert [used(graph), used(graph)] == [2, 0]                    # captured, replayed
    hub.set_vector_potential([0.1, 0.0, 0.0])
    assert [used(x) for x in calls] == [0, 0, 0]
    hub.set_vector_potential(None)
    hub.set_worklist(False)
    assert [used(x) for x in calls] == [0, 0, 0]
    hub.set_worklist(True)
    assert [used(x) for x in calls] == [1, 1, 1]
    hub.close()


def test_contexts_without_the_list():
    for kw in (dict(rc=0.4), dict(spin="unpolarized", is_complex=False)):      # one pass; real states
        hub = _context(**kw)
        assert hub.query(17) == 0
        hub.project(_inputs(hub, 48)[0])
        assert hub.query(18) == 0
        hub.close()


@pytest.mark.parametrize("spin,states", [("collinear", 64), ("collinear", 13), ("spinor", 24)])
def test_apply_keeps_no_workspace(spin, states):
    hub = _context(spin=spin)
    psi, f = _inputs(hub, states)
    c = hub.project(psi)
    n, _, _ = hub.occupations(c, f)
    ueff = [torch.full((hub.nsites,), u, dtype=torch.float64, device="cuda") for u in (0.3, -0.4)]
    # a field's apply allocates the row that padding entries write, all that an apply needs
    hub.set_vector_potential([0.0, 0.0, 0.0])
    hub.apply(ueff[0], n, c, torch.zeros_like(psi))
    hub.set_vector_potential(None)
    allocations, taken = hub.query(15), hub.query(18)
    ref = [torch.zeros_like(psi) for _ in ueff]
    for u, h in zip(ueff, ref):
        hub.apply(u, n, c, h)
    assert hub.query(15) == allocations and hub.query(18) == taken + 2
    # two potentials on all sets, and two halves of the sets, on two streams at once
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    half = [c[:1].contiguous(), c[1:].contiguous()]
    for _ in range(10):
        h = [torch.zeros_like(psi) for _ in ueff]
        g = torch.zeros_like(psi)
        torch.cuda.synchronize()
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                hub.apply(ueff[i], n, c, h[i])
                hub.apply(ueff[0], n, half[i], g[:1] if i == 0 else g[1:], sets=(i, 1 if i == 0 else hub.nsets - 1))
        torch.cuda.synchronize()
        assert torch.equal(h[0], ref[0]) and torch.equal(h[1], ref[1]) and torch.equal(g, ref[0])
    hub.close()


def test_finalize_does_without_the_list_when_memory_runs_out(monkeypatch):
    """Every allocation of hub_finalize fails once: either the call reports
    it and succeeds when repeated, or it was one of the list's and the context
    runs the passes."""
    ref = _context()
    psi, f = _inputs(ref, 40)
    taken = ref.step(psi, f, torch.zeros_like(psi), mode="batched")["c"]
    ref.set_vector_potential([0.0, 0.0, 0.0])
    passes = ref.step(psi, f, torch.zeros_like(psi), mode="batched")["c"]
    hub = _context()
    total, bytes_with = hub.query(15), hub.query(9)
    hub.close()
    without = []
    for i in range(1, total + 1):
        print(f"[fail-alloc] attempt {i} of {total}", flush=True)
        monkeypatch.setenv("HUB_FAIL_ALLOC", str(i))
        hub = _context(finalize=False)
        monkeypatch.delenv("HUB_FAIL_ALLOC")
        try:
            hub.finalize()
            # not met: only the list's own failures are passed over
            assert hub.query(17) == 0
            without.append(hub.query(9))
        except H.HubError as e:
            assert e.code == H.HUB_ENOMEM
            hub.finalize()
            assert hub.query(17) == 1 and hub.query(9) == bytes_with
        used = hub.query(18)
        c = hub.step(psi, f, torch.zeros_like(psi), mode="batched")["c"]
        assert hub.query(18) - used == (2 if hub.query(17) else 0)
        # the sums of a vanishing field's passes, whose phases are formed on the GPU
        assert (torch.equal(c, taken) if hub.query(17) else (c - passes).abs().max() < 1e-12 * passes.abs().max())
        hub.close()
    # its lists, tables and the covers that these are made from; all released
    assert len(without) == 13 and len(set(without)) == 1 and without[0] < bytes_with
    ref.close()


@pytest.fixture(scope="module")
def crystal():
    """Rocksalt cell of 44^3 points whose second pass covers 6 % of them, 8 k-points."""
    a = 8.35
    sites = [dict(R=[x * a for x in p], l=l, zeta=z, rc=rc, species=t)
             for p, l, z, rc, t in [((0, 0, 0), 2, 2.2, 4.83, 0), ((.5, .5, .5), 2, 2.2, 4.83, 0),
                                    ((.5, .5, 0), 1, 1.6, 4.025, 1), ((0, 0, .5), 1, 1.6, 4.025, 1)]]
    kpts = [[x, y, z] for x in (-.25, .25) for y in (-.25, .25) for z in (-.25, .25)]
    hub = H.Hubbard((a, a, a), (44, 44, 44), sites, kpts=kpts, kweights=[0.125] * 8, spin="collinear",
                    is_complex=True, precision="f32")
    assert hub.query(14) == 2 and hub.query(17) == 1
    yield hub
    hub.close()


@pytest.mark.parametrize("states,ld,project,apply", [
    (8, 8, 0, 1),          # narrow rows: the projection would read more table than rows, the apply's lanes idle
    (33, 33, 0, 0),        # rows that start anywhere: the tiles' lines are read and written twice
    (33, 48, 0, 1),        # the same columns on whole lines
])
def test_route_follows_what_the_rows_cost(crystal, states, ld, project, apply):
    hub = crystal
    gen = torch.Generator(device="cuda").manual_seed(ld)
    base = torch.randn((hub.nsets, hub.G, ld), generator=gen, device="cuda", dtype=hub.state_dtype)
    psi = base[:, :, :states]
    f = torch.rand((hub.nsets, states), generator=gen, device="cuda", dtype=torch.float64)
    before = hub.query(18)
    c = hub.project(psi)
    assert hub.query(18) - before == project
    n, _, _ = hub.occupations(c, f)
    ueff = torch.full((hub.nsites,), 0.2, dtype=torch.float64, device="cuda")
    h = base.clone()
    before = hub.query(18)
    hub.apply(ueff, n, c, h[:, :, :states])
    assert hub.query(18) - before == apply
    assert torch.equal(h[:, :, states:], base[:, :, states:])
    # either route gives the passes' sums: up to three FP32 roundings of a component apart
    hub.set_vector_potential([0.0, 0.0, 0.0])
    ref = base.clone()
    hub.apply(ueff, n, c, ref[:, :, :states])
    c2 = hub.project(psi)
    hub.set_vector_potential(None)
    assert (c - c2).abs().max() < 1e-13 * c2.abs().max() * 10
    assert (h - ref).abs().max() < 2.6e-7 * ref.abs().max()
