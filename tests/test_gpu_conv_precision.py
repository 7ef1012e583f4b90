"""Weight and bias gradient of wide layers over many pixels, where a workgroup
adds hundreds of pixel blocks: no further from 64 bits than FP32 sums over short
slices (dn_conv3x3_wgrad) and PyTorch's FP32 sum are."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(4, 224, 128, 256, 256), (16, 112, 48, 256, 256), (16, 96, 96, 256, 256),
                                   (12, 160, 64, 250, 255)])
def test_error_against_64_bits(shape):
    import torch
    import torch.nn.functional as F
    from paper_1608_05238_amd import _lib as L
    from paper_1608_05238_amd import denoise as D
    n, ci, co, h, w = shape
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(n, ci, h, w, generator=g, device="cuda").relu_()
    gy = torch.randn(n, co, h, w, generator=g, device="cuda")
    wt = torch.zeros(co, ci, 3, 3, device="cuda", requires_grad=True)
    b = torch.zeros(co, device="cuda", requires_grad=True)
    gw, gb = torch.autograd.grad(D.conv3x3(x, wt, b), (wt, b), gy)
    xb, gyb = x.to(torch.bfloat16), gy.to(torch.bfloat16)
    ref = torch.zeros(co, ci, 3, 3, dtype=torch.float64, device="cuda")
    for i in range(n):   # products of BF16 values in 64 bits, one image and tap at a time
        xp, gi = F.pad(xb[i].double(), (1, 1, 1, 1)), gyb[i].double().reshape(co, h * w)
        for t in range(9):
            part = xp[:, t // 3:t // 3 + h, t % 3:t % 3 + w].reshape(ci, h * w)
            ref[:, :, t // 3, t % 3] += gi @ part.t().contiguous()
    xl, gl = (v.permute(0, 2, 3, 1).contiguous() for v in (xb, gyb))
    short = torch.empty(co, 3, 3, ci, device="cuda")
    L.check("dn_conv3x3_wgrad", L.load().dn_conv3x3_wgrad(xl.data_ptr(), gl.data_ptr(), short.data_ptr(), n, ci, co, h, w,
                                                          C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    err = lambda a, r: float((a.double() - r).norm() / r.norm())
    assert err(gw, ref) <= err(short.permute(0, 3, 1, 2), ref), shape
    assert err(gb, gy.double().sum((0, 2, 3))) <= err(gy.sum((0, 2, 3)), gy.double().sum((0, 2, 3))), shape
