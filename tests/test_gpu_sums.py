"""Sums over the pixels (mc_residual's eps, mc_detect) around the sizes where
the number of workgroups and the pixels per thread change, against NumPy; the
same bits again and on several streams at once."""
import math

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _inputs(nz, nx, N, seed=0):
    import torch
    from paper_1608_05238_amd import rmc
    rng = np.random.default_rng(seed)
    K = 2 * N + 1
    a = {"mua": rng.uniform(0.01, 0.1, (nz, nx)).astype(np.float32), "f": rng.standard_normal((K, nz, nx)),
         "d": rng.standard_normal((K, nz, nx)), "h": rng.standard_normal((nz, nx))}
    t = {k: torch.as_tensor(v, device="cuda") for k, v in a.items()}
    return a, t, rmc.Medium(t["mua"], t["mua"] * 100, t["mua"], 0.1)


@pytest.mark.parametrize("shape", [(1, 1, 0), (1, 255, 1), (16, 16, 2), (1, 257, 3), (255, 257, 2), (256, 256, 16),
                                   (1, 65537, 0), (300, 450, 4)])
def test_sums_against_numpy(shape):
    import torch
    from paper_1608_05238_amd import rmc
    nz, nx, N = shape
    a, t, med = _inputs(nz, nx, N)
    area = float(np.float32(0.1)) ** 2
    mua = a["mua"].astype(np.float64)
    r = a["h"] - mua * a["f"][0]
    q, eps = rmc.mc_residual(med, t["f"], t["h"])
    # n terms in any order: below n 2^-53 of the sum of magnitudes, n <= 2^17
    assert float(eps) == pytest.approx(0.5 * area * math.fsum((r * r).ravel()), rel=2e-11)
    assert np.allclose(q.cpu().numpy(), mua * r, rtol=1e-13, atol=1e-15)
    w = np.full((2 * N + 1, 1, 1), 1 / math.pi)
    w[0] = 0.5 / math.pi
    terms = (a["f"] * a["d"] * w).ravel() * area
    out = rmc.mc_detect(med, N, t["f"], t["d"])
    assert abs(float(out) - math.fsum(terms)) <= 2e-11 * np.abs(terms).sum()
    for _ in range(3):
        assert float(rmc.mc_detect(med, N, t["f"], t["d"])) == float(out)
        assert torch.equal(rmc.mc_residual(med, t["f"], t["h"])[1], eps)


def test_sums_on_many_streams():
    """More calls in flight than the pool of parts has slots."""
    import torch
    from paper_1608_05238_amd import rmc
    _, t, med = _inputs(200, 300, 8)
    ref = float(rmc.mc_detect(med, 8, t["f"], t["d"]))
    e = float(rmc.mc_residual(med, t["f"], t["h"])[1])
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(8)]
    got = []
    for i in range(240):
        with torch.cuda.stream(streams[i % 8]):
            got.append((rmc.mc_detect(med, 8, t["f"], t["d"]), rmc.mc_residual(med, t["f"], t["h"])[1]))
    torch.cuda.synchronize()
    assert all(float(x) == ref and float(y) == e for x, y in got)
