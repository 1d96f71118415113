"""hub_coulomb with an output tensor: the tensor is complete when the call
returns, for a reader on any stream."""

import pytest
import torch

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_1711_08935_amd as H  # noqa: E402


def test_tensor_is_complete_on_return():
    hub = H.Hubbard((8.0,) * 3, (16,) * 3, [dict(R=(4.0, 4.1, 3.9), l=3, zeta=1.5, rc=3.0, species=0)],
                    spin="unpolarized", is_complex=False, precision="f64")
    hub.coulomb(0)
    torch.cuda.synchronize()
    other = torch.cuda.Stream()
    for _ in range(50):
        t = hub.coulomb(0)
        assert torch.cuda.current_stream().query()                 # nothing of the call is left to run
        with torch.cuda.stream(other):
            copy = t.clone()
        other.synchronize()
        assert torch.equal(copy, hub.get_coulomb(0))
    hub.close()
