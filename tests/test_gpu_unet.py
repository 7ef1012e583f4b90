"""The denoiser's network without gradients (one call of dn_unet_forward)
against the same network layer by layer.  Its maps are the same bits up to the
output layer, so with one weight per output row (a product, no sum) the results
are too; with all weights the FP32 sums of c terms differ by their order only:
2 c 2^-24 of the sum of magnitudes, plus the roundings of bias and x."""
import pytest

pytestmark = pytest.mark.gpu


def _mods():
    import torch
    import torch.nn.functional as F
    from paper_1608_05238_amd import denoise as D
    return torch, F, D


def _by_layers(torch, F, model, x):
    """(result, input of the output layer)"""
    with torch.no_grad():
        h, skips = x, []
        for i, (c1, c2) in enumerate(model.enc):
            h = F.relu(c2(F.relu(c1(h))))
            if i < len(model.enc) - 1:
                skips.append(h)
                h = F.max_pool2d(h, 2, ceil_mode=True)
        for c1, c2 in model.dec:
            s = skips.pop()
            h = F.interpolate(h, scale_factor=2, mode="nearest")[:, :, :s.shape[2], :s.shape[3]]
            h = F.relu(c2(F.relu(c1(torch.cat([h, s], 1)))))
        corr = torch.einsum("oc,nchw->nohw", model.out, h) + model.out_bias[None, :, None, None]
        return x + corr, h


def _model(torch, D, channels, widths, seed):
    torch.manual_seed(seed)
    model = D.UNet(channels, widths=widths).cuda()
    with torch.no_grad():
        for c in model._layers():
            c.bias.normal_(0, 0.1)
        model.out.normal_(0, 0.3)
        model.out_bias.normal_(0, 0.1)
    return model


@pytest.mark.parametrize("case", [(33, (24, 32, 48), 3, 64, 64), (5, (16, 24), 2, 37, 50), (9, (8,), 1, 17, 5),
                                  (3, (20, 12, 33), 2, 41, 23), (1, (48, 64, 96, 64), 1, 9, 1), (7, (8, 8, 8, 8), 1, 1, 3),
                                  (33, (24, 32, 48, 64, 96, 128), 1, 130, 258), (2, (130, 16), 2, 20, 20)])
def test_one_call_equals_the_layers(case):
    torch, F, D = _mods()
    channels, widths, n, h, w = case
    model = _model(torch, D, channels, widths, sum(widths))
    x = torch.randn(n, channels, h, w, device="cuda")
    wide = torch.randn(n, channels + 2, h, w + 1, device="cuda")
    for xf in (x, x.contiguous(memory_format=torch.channels_last), wide[:, 1:-1, :, 1:]):
        want, a = _by_layers(torch, F, model, xf)
        with torch.no_grad():
            assert model._plain(xf) and model._inference(xf) is not None
            got = model(xf)
        assert got.stride() == want.stride()
        bound = (2 * widths[0] * 2.0 ** -24 * torch.einsum("oc,nchw->nohw", model.out.abs().double(), a.abs().double())
                 + 2.0 ** -22 * (want.abs() + xf.abs() + 1.0))
        assert bool(((got.double() - want.double()).abs() <= bound).all())
    with torch.no_grad():
        keep = torch.randint(widths[0], (channels, 1), device="cuda")
        model.out.copy_(torch.zeros_like(model.out).scatter_(1, keep, 0.7))
        want, _ = _by_layers(torch, F, model, x)
        assert torch.equal(model(x), want)
        x[0, 0, h // 2, w // 2] = float("nan")   # goes through ReLU and maxima
        want, _ = _by_layers(torch, F, model, x)
        assert torch.equal(model(x).isnan(), want.isnan())


def test_what_has_to_see_the_layers_does():
    """Gradients, hooks, replaced layers, other types and shapes take the layers one by one."""
    torch, F, D = _mods()
    model = _model(torch, D, 4, (8, 16), 0)
    x = torch.randn(2, 4, 12, 12, device="cuda")
    assert not model._plain(x)
    with torch.no_grad():
        assert model._plain(x)
        assert not model._plain(x.double()) and not model._plain(x[:, :3]) and not model._plain(x.cpu())
        with torch.autocast("cuda", dtype=torch.bfloat16):
            assert not model._plain(x)
        with torch.autograd.forward_ad.dual_level():
            assert not model._plain(x)
        seen = []
        hook = model.enc[1][0].register_forward_hook(lambda m, i, o: seen.append(o.shape))
        model(x)
        assert len(seen) == 1
        hook.remove()
        model.dec[0][1] = torch.nn.Conv2d(8, 8, 3, padding=1).cuda()
        assert not model._plain(x)
        model(x)
        deep = _model(torch, D, 4, (8,) * 9, 0)   # more levels than one call takes
        assert deep._plain(x) and deep._inference(x) is None
        want, _ = _by_layers(torch, F, deep, x)
        assert torch.equal(deep(x), want)


def test_one_call_under_graph_capture():
    torch, F, D = _mods()
    model = _model(torch, D, 5, (16, 24), 1)
    x = torch.randn(2, 5, 33, 40, device="cuda")
    with torch.no_grad():
        model(x)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            y = model(x)
        for i in range(3):
            x.normal_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, model(x))
