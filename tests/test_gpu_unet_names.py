"""The network without gradients when PyTorch lacks the names by which it tells
whether something has to see the layers: they run one by one."""
import types

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("module", ["forward_ad", "nn_module"])
def test_missing_names_mean_layer_by_layer(module, monkeypatch):
    import torch
    from paper_1608_05238_amd import denoise as D
    torch.manual_seed(0)
    model = D.UNet(5, (8, 16)).cuda()
    x = torch.randn(1, 5, 12, 14, device="cuda")
    with torch.no_grad():
        assert model._plain(x)
        want = model(x)
        monkeypatch.setattr(D, module, types.SimpleNamespace())
        assert not model._plain(x)
        assert torch.equal(model(x), want)   # the output layer is zero: the same bits
