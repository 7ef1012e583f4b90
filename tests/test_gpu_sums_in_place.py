"""mc_residual and mc_detect where an output lies in an input: q* over the
measured map or the a0 plane, and the sum's eight bytes inside a map.  The same
bits as with outputs of their own."""
import ctypes as C

import pytest

from .test_gpu_sums import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 5), (16, 16), (31, 33), (255, 257)])
def test_outputs_inside_inputs(shape):
    import torch
    from paper_1608_05238_amd import _lib as L, rmc
    lib, N = L.load(), 2
    _, t, med = _inputs(*shape, N)
    m, s = med.c(), C.c_void_p(torch.cuda.current_stream().cuda_stream)
    q, eps = rmc.mc_residual(med, t["f"], t["h"])
    det = rmc.mc_detect(med, N, t["f"], t["d"])

    def residual(where, spot):
        """q* into a copy of `where`, eps into its own word or into element `spot` of a map."""
        f, h = t["f"].clone(), t["h"].clone()
        out = {"h": h, "a0": f[0], "own": torch.empty_like(h), None: None}[where]
        e = torch.zeros(1, dtype=torch.float64, device="cuda") if spot is None else \
            {"h": h, "a0": f[0], "q": out}[spot[0]].view(-1)[spot[1]:][:1]
        L.check("mc_residual", lib.mc_residual(C.byref(m), f.data_ptr(), h.data_ptr(), None if out is None else
                                               out.data_ptr(), e.data_ptr(), s))
        return out, e[0].clone()

    last = shape[0] * shape[1] - 1
    for where in ("h", "a0", "own"):
        out, e = residual(where, None)
        assert torch.equal(out, q) and torch.equal(e, eps), where
        for spot in (("h", 0), ("a0", last), ("q", last // 2)):
            out, e = residual(where, spot)
            assert torch.equal(e, eps), (where, spot)
            same = out == q
            if spot[0] == "q" or spot[0] == where:   # eps is written last, over one value
                same.view(-1)[spot[1]] = True
            assert bool(same.all()), (where, spot)
    assert torch.equal(residual(None, None)[1], eps) and torch.equal(residual(None, ("h", last))[1], eps)
    for key in ("f", "d"):
        c = {k: t[k].clone() for k in ("f", "d")}
        out = c[key].view(-1)[last:][:1]
        L.check("mc_detect", lib.mc_detect(C.byref(m), N, c["f"].data_ptr(), c["d"].data_ptr(), out.data_ptr(), s))
        assert torch.equal(out[0], det), key
