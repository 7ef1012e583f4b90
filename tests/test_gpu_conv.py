"""The convolution kernels over what their launch plan chooses between: 16 x 16
and 8 x 8 pixel blocks, 16 to 64 output channels a workgroup, channels in one
piece or several, activations read as whole 16-byte units or element by
element.  Values against FP64 on the same BF16-rounded operands (the products
are exact in FP32; only the order of the FP32 sums differs: the bound is that
of tests/test_gpu_denoise.py); the ways of reading an activation against each
other, bit for bit, as all of them add in the same order."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


def _mods():
    import torch
    import torch.nn.functional as F
    from paper_1608_05238_amd import _lib as L
    from paper_1608_05238_amd import denoise as D
    return torch, F, L, D


# (n, ci, co, h, w)
SHAPES = [(2, 8, 16, 249, 250),      # 16 output channels, one unit
          (2, 24, 30, 250, 249),     # 32, rows of the result not in 16 bytes
          (2, 33, 48, 241, 256),     # 48, padded input channels
          (2, 72, 64, 241, 241),     # 64, input channels in three pieces
          (2, 50, 20, 256, 241),     # two pieces, whole units short of the last
          (1, 40, 63, 178, 177),     # 144 blocks of 16 x 16, 32 channels a workgroup
          (1, 16, 16, 511, 16),      # 32 blocks of 16 x 16 would be too few: 8 x 8
          (1, 128, 128, 8, 8),       # fewer channels a workgroup
          (3, 56, 49, 15, 17),       # edges of 8 x 8 blocks, odd output channels
          (1, 9, 1, 1, 40)]


@pytest.mark.parametrize("shape", SHAPES)
def test_conv_values_layouts_and_gradients(shape):
    torch, F, L, D = _mods()
    n, ci, co, h, w = shape
    g = torch.Generator().manual_seed(sum(shape))
    x = torch.randn(n, ci, h, w, generator=g)
    wt = torch.randn(co, ci, 3, 3, generator=g) / (3 * ci ** 0.5)
    b = torch.randn(co, generator=g)
    gy = torch.randn(n, co, h, w, generator=g)
    xr, wr, gyr = (t.to(torch.bfloat16).double() for t in (x, wt, gy))
    xr.requires_grad_(True)
    wr.requires_grad_(True)
    yr = F.conv2d(xr, wr, b.double(), padding=1)
    yr.backward(gyr)
    ref = (yr.detach(), xr.grad, wr.grad, gy.double().sum((0, 2, 3)))

    wd, bd = wt.cuda().requires_grad_(True), b.cuda().requires_grad_(True)
    xc = x.cuda()
    wide = torch.zeros(n, ci + 3, h, w, device="cuda").contiguous(memory_format=torch.channels_last)
    wide[:, 1:ci + 1] = xc
    forms = {"planes": xc, "rows": xc.contiguous(memory_format=torch.channels_last),
             "turned": xc.transpose(2, 3).contiguous().transpose(2, 3), "part of wider rows": wide[:, 1:ci + 1]}
    gforms = {"planes": gy.cuda(), "rows": gy.cuda().contiguous(memory_format=torch.channels_last)}
    first = None
    for name, xf in forms.items():
        for gname, gf in gforms.items():
            leaf = xf.detach().requires_grad_(True)
            wd.grad = bd.grad = None
            y = D.conv3x3(leaf, wd, bd)
            y.backward(gf)
            got = [t.detach() for t in (y, leaf.grad, wd.grad, bd.grad)]
            if first is None:
                first = got
                for a, r in zip(got, ref):
                    err = float((a.double().cpu() - r).abs().max() / r.abs().max().clamp_min(1e-30))
                    assert err < 2e-5, (shape, tuple(r.shape), err)
            for a, f in zip(got, first):
                assert torch.equal(a, f), (shape, name, gname, tuple(a.shape))
        with torch.no_grad():
            assert torch.equal(D.conv3x3(xf, wd, bd), first[0]), (shape, name)

    # the entry for BF16 operands: the same result from operands rounded before
    lib, cip = L.load(), (ci + 7) // 8 * 8
    xb = F.pad(xc.to(torch.bfloat16).permute(0, 2, 3, 1), (0, cip - ci)).contiguous()
    wb = F.pad(wt.cuda().to(torch.bfloat16).permute(0, 2, 3, 1), (0, cip - ci)).contiguous()
    y = torch.empty(n, h, w, co, device="cuda")
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    L.check("dn_conv3x3_fwd", lib.dn_conv3x3_fwd(xb.data_ptr(), wb.data_ptr(), bd.data_ptr(), y.data_ptr(), n, cip, co,
                                                 h, w, s))
    assert torch.equal(y.permute(0, 3, 1, 2), first[0])


def test_repeated_rows_and_one_value_gradient():
    """An expanded activation (strides of zero) and an expanded upstream gradient."""
    torch, F, L, D = _mods()
    torch.manual_seed(1)
    row = torch.randn(1, 12, 1, 20, device="cuda")
    wd = torch.randn(10, 12, 3, 3, device="cuda", requires_grad=True)
    bd = torch.zeros(10, device="cuda", requires_grad=True)
    res = []
    for x in (row.expand(2, 12, 14, 20), row.expand(2, 12, 14, 20).contiguous()):
        wd.grad = bd.grad = None
        y = D.conv3x3(x, wd, bd)
        y.sum().backward()
        res.append((y.detach(), wd.grad, bd.grad))
    for a, b in zip(*res):
        assert torch.equal(a, b)
    assert torch.equal(res[0][2], torch.full((10,), 2.0 * 14 * 20, device="cuda"))


def test_gradients_refuse_small_or_missing_scratch():
    torch, F, L, D = _mods()
    lib = L.load()
    need = lib.dn_conv3x3_grads_bytes(1, 16, 16, 16, 16)
    assert need > 0 and lib.dn_conv3x3_grads_bytes(0, 16, 16, 16, 16) == 0
    x = torch.zeros(1, 16, 16, 16, device="cuda", dtype=torch.bfloat16)
    g, gw = torch.zeros(1, 16, 16, 16, device="cuda"), torch.zeros(16, 16, 3, 3, device="cuda")
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)
    call = lambda ptr, size: lib.dn_conv3x3_grads(x.data_ptr(), g.data_ptr(), gw.data_ptr(), None, ptr, size, 1, 16, 16, 16,
                                                  16, s)
    assert call(ws.data_ptr(), need - 1) != 0 and call(None, need) != 0
    assert call(ws.data_ptr(), need) == 0
