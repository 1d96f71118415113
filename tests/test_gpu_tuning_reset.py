"""A tuned context returns to the automatic kernel shapes: hub_set_tuning with
(0, 0, -1) gives the bits of a context that was never tuned."""

import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402
from tests.gpu_common import device_states, make_hub, states_and_occupations  # noqa: E402
from synth import make_config  # noqa: E402


def test_reset_to_automatic():
    cfg = make_config("nio_afm", small=True)
    psi, f = states_and_occupations(cfg)
    hubs = [make_hub(cfg, "f64", chunk=256) for _ in range(2)]
    psi_d, _ = device_states(hubs[0], psi)
    f_d = torch.from_numpy(f).cuda()
    out = []
    for tune, hub in enumerate(hubs):
        for i in range(hub.nsites):
            hub.set_fixed_ueff(i, 0.2)
        if tune:
            for which in (0, 1):
                hub.set_tuning(which, 1, 1, 1)
            hub.step(psi_d, f_d, torch.zeros_like(psi_d), mode="batched")
            for which in (0, 1):
                hub.set_tuning(which, 0, 0, -1)
        h = torch.zeros_like(psi_d)
        out.append((hub.step(psi_d, f_d, h, mode="batched"), h))
    for k in ("c", "n", "U"):
        assert torch.equal(out[0][0][k], out[1][0][k]), k
    assert torch.equal(out[0][1], out[1][1])
    for bad in (-1, 3, 8):
        with pytest.raises(H.HubError) as e:
            hubs[0].set_tuning(0, 0, bad)
        assert e.value.code == H.HUB_EINVAL
    for hub in hubs:
        hub.close()
