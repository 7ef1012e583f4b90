"""Which networks the denoiser's one call may take, without a GPU: a stand-in
for the library records whether it would have been called."""
import pytest


class _Lib:
    def __init__(self):
        self.calls = []

    def dn_unet_bytes(self, ch, levels, widths, n, h, w):
        return 1024

    def dn_unet_forward(self, ch, levels, widths, weights, biases, *rest):
        self.calls.append((levels, len(weights), len(biases)))
        return 0


@pytest.fixture
def lib(monkeypatch):
    from paper_1608_05238_amd import denoise as D
    lib = _Lib()
    monkeypatch.setattr(D.L, "load", lambda: lib)
    monkeypatch.setattr(D, "_stream", lambda: None)
    return lib


def test_a_decoder_of_another_length_is_left_to_the_layers(lib):
    """The call reads the pointers of 4 levels - 2 layers: a network with fewer
    or more decoder levels than its encoder has must not reach it."""
    import torch
    from paper_1608_05238_amd import denoise as D
    x = torch.randn(1, 5, 12, 12)
    model = D.UNet(5, widths=(8, 16, 24))
    assert model._inference(x) is not None and lib.calls == [(3, 10, 10)]
    for dec in (model.dec[:1], model.dec[:0], [*model.dec, model.dec[1]]):
        other = D.UNet(5, widths=(8, 16, 24))
        other.dec = torch.nn.ModuleList(dec)
        assert other._inference(x) is None
    assert D.UNet(5, widths=())._inference(x) is None   # no level at all: the output layer alone
    assert len(lib.calls) == 1
