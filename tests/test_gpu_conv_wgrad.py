"""dn_conv3x3_wgrad, the weight gradient from BF16 operands without scratch
memory, against FP64 on the same operands (the products are exact in FP32; only
the order of the FP32 sums differs: the bound of tests/test_gpu_denoise.py),
and the convolution benchmark, which times what a layer calls."""
import ctypes as C

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 8, 8, 1, 1), (2, 24, 40, 9, 17), (1, 40, 72, 33, 31), (3, 64, 64, 64, 64)])
def test_weight_gradient_values(shape):
    import torch
    import torch.nn.functional as F
    from paper_1608_05238_amd import _lib as L
    n, ci, co, h, w = shape
    g = torch.Generator().manual_seed(sum(shape))
    x, gy = (torch.randn(n, c, h, w, generator=g).to(torch.bfloat16) for c in (ci, co))
    wt = torch.zeros(co, ci, 3, 3, dtype=torch.float64, requires_grad=True)
    F.conv2d(x.double(), wt, padding=1).backward(gy.double())
    xd, gd = (t.cuda().permute(0, 2, 3, 1).contiguous() for t in (x, gy))
    gw = torch.full((co, 3, 3, ci), float("nan"), device="cuda")
    L.check("dn_conv3x3_wgrad", L.load().dn_conv3x3_wgrad(
        xd.data_ptr(), gd.data_ptr(), gw.data_ptr(), n, ci, co, h, w, C.c_void_p(torch.cuda.current_stream().cuda_stream)))
    err = float((gw.permute(0, 3, 1, 2).double().cpu() - wt.grad).abs().max() / wt.grad.abs().max())
    assert err < 2e-5, (shape, err)


def test_benchmark_times_the_layer_s_entry_points(monkeypatch):
    from paper_1608_05238_amd import _lib as L
    from paper_1608_05238_amd import denoise as D
    lib, called = L.load(), set()

    class Recorder:
        def __getattr__(self, name):
            called.add(name)
            return getattr(lib, name)

    monkeypatch.setattr(D.L, "load", lambda: Recorder())
    rows = D.conv_bench(reps=1)["rows"]
    assert called == {"dn_pack_weights", "dn_conv3x3_f32", "dn_conv3x3_grads_bytes", "dn_conv3x3_grads"}
    assert all(r["fwd_ms"] > 0 and r["wgrad_ms"] > 0 for r in rows)
