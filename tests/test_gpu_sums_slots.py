"""Sums over the pixels with every slot for their parts taken: the first
workgroup computes all parts, and no other one may take the sum for a slot.

A call is two kernels, of which the first takes a slot and the second gives it
back.  The test captures a call and takes one of its two nodes out: the graph
of the first alone holds a slot, that of the second alone, started from the
bytes that the first left, gives it back."""
import ctypes as C

import pytest

from .test_gpu_sums import _inputs

pytestmark = pytest.mark.gpu


def _hip():
    with open("/proc/self/maps") as f:
        path = next(line.split()[-1] for line in f if "libamdhip64" in line)
    return C.CDLL(path)


def _half(hip, stream, call, first):
    """The captured call's first node alone, or its second; an executable graph."""
    ok = lambda rc: pytest.fail(f"HIP error {rc}") if rc else None
    graph, ex = C.c_void_p(), C.c_void_p()
    ok(hip.hipStreamBeginCapture(stream, 2))
    call()
    ok(hip.hipStreamEndCapture(stream, C.byref(graph)))
    nodes, root, n, nr = (C.c_void_p * 8)(), (C.c_void_p * 8)(), C.c_size_t(8), C.c_size_t(8)
    ok(hip.hipGraphGetNodes(graph, nodes, C.byref(n)))
    ok(hip.hipGraphGetRootNodes(graph, root, C.byref(nr)))
    assert n.value == 2 and nr.value == 1
    for i in range(2):
        if (nodes[i] == root[0]) != first:
            ok(hip.hipGraphDestroyNode(C.c_void_p(nodes[i])))
    ok(hip.hipGraphInstantiate(C.byref(ex), graph, None, None, 0))
    return ex


def test_every_slot_taken():
    import torch
    from paper_1608_05238_amd import _lib as L, rmc
    hip, lib = _hip(), L.load()
    _, t, med = _inputs(255, 257, 3)
    s = torch.cuda.Stream()
    stream = C.c_void_p(s.cuda_stream)
    want = rmc.mc_detect(med, 3, t["f"], t["d"])
    eps = rmc.mc_residual(med, t["f"], t["h"])[1]
    res = torch.zeros(1, dtype=torch.int64, device="cuda")
    m = med.c()
    call = lambda: L.check("mc_detect", lib.mc_detect(C.byref(m), 3, t["f"].data_ptr(), t["d"].data_ptr(),
                                                      res.data_ptr(), stream))
    torch.cuda.synchronize()
    take, give = _half(hip, stream, call, True), _half(hip, stream, call, False)
    held = []
    try:
        for _ in range(200):
            assert hip.hipGraphLaunch(take, stream) == 0
            torch.cuda.synchronize()
            if int(res) == 0:
                break
            held.append(int(res))
        assert len(held) == len(set(held)) >= 1 and int(res) == 0   # every slot is taken
        for _ in range(5):
            assert torch.equal(rmc.mc_detect(med, 3, t["f"], t["d"]), want)
            assert torch.equal(rmc.mc_residual(med, t["f"], t["h"])[1], eps)
    finally:
        for tag in held:
            res.fill_(tag)
            torch.cuda.synchronize()
            assert hip.hipGraphLaunch(give, stream) == 0
            torch.cuda.synchronize()
            assert torch.equal(res.view(torch.float64)[0], want)
    assert hip.hipGraphLaunch(take, stream) == 0   # there are slots again
    torch.cuda.synchronize()
    assert int(res) in held
    assert hip.hipGraphLaunch(give, stream) == 0
    torch.cuda.synchronize()
    assert torch.equal(res.view(torch.float64)[0], want)
    assert torch.equal(rmc.mc_detect(med, 3, t["f"], t["d"]), want)
