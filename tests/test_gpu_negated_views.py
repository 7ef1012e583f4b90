"""Tensors whose sign is a property of the view (the imaginary part of a
conjugate): the kernels read memory, so the sign has to be put in first."""
import pytest

pytestmark = pytest.mark.gpu


def _neg(t):
    """A view equal to t that carries the negative bit."""
    import torch
    z = torch.complex(torch.zeros_like(t), -t)
    v = z.conj().imag
    assert v.is_neg() and torch.equal(v, t)
    return v


def test_convolution_and_its_gradients():
    import torch
    from paper_1608_05238_amd import denoise as D
    torch.manual_seed(0)
    x, w, b = (torch.randn(*s, device="cuda") for s in ((2, 5, 9, 11), (6, 5, 3, 3), (6,)))
    gy = torch.randn(2, 6, 9, 11, device="cuda")
    res = []
    for neg in ((), (0,), (1,), (2,), (3,), (0, 1, 2, 3)):
        leaves = [t.detach().clone().requires_grad_(True) for t in (x, w, b)]
        a = [_neg(t) if i in neg else t for i, t in enumerate((*leaves, gy))]
        y = D.conv3x3(*a[:3])
        y.backward(a[3])
        res.append([y.detach()] + [t.grad for t in leaves])
        with torch.no_grad():
            res[-1].append(D.conv3x3(*a[:3]))
    for r in res[1:]:
        assert all(torch.equal(p, q) for p, q in zip(r, res[0]))


def test_network_without_gradients():
    import torch
    from paper_1608_05238_amd import denoise as D
    torch.manual_seed(0)
    model = D.UNet(5, (8, 16)).cuda()
    with torch.no_grad():
        model.out.normal_()
        x = torch.randn(1, 5, 12, 14, device="cuda")
        want = model(x)
        # layer by layer: the output layer's sums in another order, 2 c 2^-24 of their magnitudes, c = 8
        assert torch.allclose(model(_neg(x)), want, rtol=1e-5, atol=1e-5 * float(want.abs().max()))
