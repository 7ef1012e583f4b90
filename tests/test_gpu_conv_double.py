"""The bias gradient of a convolution is a sum of the upstream gradient: with
create_graph it stays part of the graph, whether or not the weights ask for
theirs."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weights", [True, False])
def test_bias_gradient_can_be_differentiated(weights):
    import torch
    from paper_1608_05238_amd import denoise as D
    torch.manual_seed(2)
    x = torch.randn(2, 5, 9, 11, device="cuda")
    w = torch.randn(6, 5, 3, 3, device="cuda", requires_grad=weights)
    b = torch.zeros(6, device="cuda", requires_grad=True)
    gy = torch.randn(2, 6, 9, 11, device="cuda", requires_grad=True)
    y = D.conv3x3(x, w, b)
    want = gy.detach().sum((0, 2, 3))
    ask = (w, b) if weights else (b,)
    gb = torch.autograd.grad(y, ask, gy, create_graph=True)[-1]
    # 198 FP32 terms in another order
    assert torch.allclose(gb, want, rtol=0, atol=198 * 2.0 ** -24 * float(gy.detach().abs().sum((0, 2, 3)).max()))
    g2, = torch.autograd.grad(gb.pow(2).sum(), gy)
    assert torch.equal(g2, (2 * gb.detach())[None, :, None, None].expand_as(gy))
    plain = torch.autograd.grad(D.conv3x3(x, w, b), ask, gy)
    if weights:   # the weights' gradient does not depend on it
        assert torch.equal(plain[0], torch.autograd.grad(D.conv3x3(x, w, b), ask, gy, create_graph=True)[0])
    assert not plain[-1].requires_grad
