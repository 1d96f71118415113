"""hub_step_noalloc at the edge of its scratch array, and over the
image-summed list.

A small launch shares its chunks among several work-groups, whose partial rows
take more of the scratch than whole chunks do; a step whose workspace fits with
whole chunks is not refused."""

import ctypes

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402
from tests.test_gpu_bloch_route import _context, _inputs  # noqa: E402

SCRATCH = 128 << 20


def _step(hub, psi, S, f, h, bufs):
    io = H.StepIO(psi.data_ptr(), psi.stride(1), S, f.data_ptr(), h.data_ptr(), h.stride(1), 1.0,
                  *(bufs[k].data_ptr() for k in ("c", "n", "pbar", "nbar", "U", "J", "Ueff", "status")))
    hub._stream()
    return H.lib().hub_step_noalloc(hub._ctx, ctypes.byref(io))


def test_whole_chunks_where_their_parts_do_not_fit():
    # one d shell inside the cell (one chunk, 5 rows), real states
    S, G = 8000, 125
    hub = H.Hubbard((5.0,) * 3, (5,) * 3, [dict(R=(2.5, 2.5, 2.5), l=2, zeta=1.5, rc=2.1, species=0)],
                    spin="unpolarized", is_complex=False, precision="f32")
    hub.set_fixed_ueff(0, 0.3)
    assert hub.query(5) == 1 and hub.query(10) == 5
    gen = torch.Generator(device="cuda").manual_seed(1)
    psi = torch.randn((1, G, S), generator=gen, device="cuda", dtype=torch.float32)
    f = torch.rand((1, S), generator=gen, device="cuda", dtype=torch.float64)

    def slots(n):
        return (n + 31) // 32 * 32

    # one partial row per function; 64 splits of 14 x 14 pairs of four sums; the rest: the apply's row
    ldh = SCRATCH // 8 - slots(5 * S) - slots(64 * 196 * 4)
    bufs, ref = hub.step_buffers(S), hub.step_buffers(S)
    base = torch.empty(G * (ldh + 32), device="cuda", dtype=torch.float32)
    h = base[:G * ldh].view(1, G, ldh)[:, :, :S]
    h.zero_()
    assert _step(hub, psi, S, f, h, bufs) == H.HUB_OK
    href = torch.zeros_like(psi)
    hub.step(psi, f, href, mode="batched", bufs=ref)
    torch.cuda.synchronize()
    for k in ("c", "n", "pbar", "nbar", "U", "J", "Ueff"):
        # FP64 sums of at most 64 points and 8000 states in another order
        assert (bufs[k] - ref[k]).abs().max() <= 1e-12 * ref[k].abs().max(), k
    assert (h - href).abs().max() <= 1.2e-7 * href.abs().max()
    # one row more than fits is refused
    big = base[:G * (ldh + 32)].view(1, G, ldh + 32)[:, :, :S]
    assert _step(hub, psi, S, f, big, bufs) == H.HUB_ESCRATCH
    hub.close()


@pytest.mark.parametrize("spin,states", [("collinear", 48), ("collinear", 5), ("spinor", 20)])
def test_image_summed_list(spin, states):
    hub = _context(spin=spin, prec="f32")
    assert hub.query(17) == 1
    psi, f = _inputs(hub, states)
    bufs, ref = hub.step_buffers(states), hub.step_buffers(states)
    h, href = torch.zeros_like(psi), torch.zeros_like(psi)
    allocations, taken = hub.query(15), hub.query(18)
    hub.step_noalloc(psi, f, h, bufs)
    assert hub.query(15) == allocations and hub.query(18) == taken + 2
    hub.step(psi, f, href, mode="batched", bufs=ref)
    torch.cuda.synchronize()
    assert torch.equal(h, href) and np.isfinite(ref["c"].abs().max().item())
    for k in ("c", "n", "pbar", "nbar", "U", "J", "Ueff", "status"):
        assert torch.equal(bufs[k], ref[k]), k
    hub.close()
