"""The band gradients that autograd hands to bands of another device than the
solve's are tensors of their own (the meta device stands in for the other
device on the CPU): no band's gradient holds or resizes another's memory."""
import pytest
import torch

from paper_2107_05395_amd.autograd import _band_grads


@pytest.mark.parametrize("nb", [3, 5])
def test_each_band_on_another_device_owns_its_gradient(nb):
    n = 7
    gb = torch.arange(nb * n, dtype=torch.float64).reshape(nb, n)
    out = _band_grads(gb, [torch.device("meta")] * nb)
    for t in out:
        assert t.device.type == "meta" and t.shape == (n,) and t.dtype == torch.float64
        assert t.storage_offset() == 0 and t.untyped_storage().nbytes() == n * 8
    # bands on the solve's device take its rows; mixed devices keep the order
    out = _band_grads(gb, [torch.device("cpu")] * (nb - 1) + [torch.device("meta")])
    for q in range(nb - 1):
        assert torch.equal(out[q], gb[q])
    assert out[-1].device.type == "meta"
