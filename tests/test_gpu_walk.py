"""The walk-and-tally rounds (few packets, and the last packets of a large run)
against the generations of the tile kernel on the same packets: bitwise equal
maps and equal event counts.  A pool smaller than the run (`live_packets`)
makes the generations launch and move the packets; without it a run of this
size walks from its launch."""
import numpy as np
import pytest

import phantoms as P

pytestmark = pytest.mark.gpu

COUNTS = ("packets", "segments", "visits", "scatters")


def _run(ph, specs, n, N, adjoint=False, tuning=None, flags=0, w_th=1e-4, m=10.0, noalloc=False):
    from paper_1608_05238_amd import rmc
    med = rmc.Medium.from_phantom(ph)
    run = rmc.make_run(n, N, seed=7, stream_tag=int(adjoint), flags=flags, w_threshold=w_th, roulette_m=m)
    if noalloc:
        co, led = rmc.mc_run_noalloc(med, specs, run, adjoint, tuning=tuning)
    else:
        co, led = (rmc.mc_adjoint if adjoint else rmc.mc_forward)(med, specs, run, tuning=tuning)
    return co.cpu().numpy(), rmc.ledger_dict(led)


def _same(a, b):
    assert np.isfinite(a[0]).all() and np.array_equal(a[0], b[0]), np.abs(a[0] - b[0]).max()
    for k in COUNTS:
        assert a[1][k] == b[1][k], (k, a[1][k], b[1][k])
    for k in ("absorbed", "escaped"):
        assert a[1][k] == pytest.approx(b[1][k], rel=1e-6, abs=1e-9)


@pytest.mark.parametrize("case", ["disc", "coarse", "dense", "strip", "roulette", "truncated", "map", "equal_count"])
@pytest.mark.parametrize("tuning", [{}, {"tile": 3}, {"max_generations": 1}])
def test_rounds_equal_generations(case, tuning):
    """coarse: hundreds of segments per visit, so visits span runs and rounds;
    strip: a grid narrower than a tile; tile 3: runs of a few events;
    max_generations 1: one round, then the finisher takes the packets and the
    open visits."""
    n, N, adj, kw = 20_000, 16, False, {}
    ph = P.disc_phantom(50, 0.2, 0.02, 8.0, 0.9, seed=3, radius=(1.0, 2.0))
    specs = P.four_side_lines(ph)
    if case == "coarse":
        ph = P.homogeneous(5, 4, 8.0, 0.002, 20.0, 0.3)
        specs = [P.point_source(13.0, 15.0)]
        n, N = 300, 3
    elif case == "dense":   # absorption past the series of the absorbed fraction
        ph = P.homogeneous(40, 40, 0.5, 1.5, 3.0, 0.5)
        specs = P.lambertian_boundary(ph)
    elif case == "strip":
        ph = P.homogeneous(3, 90, 0.3, 0.01, 5.0, 0.8)
        specs = P.pencil_top_centre(ph)
        N = 32
    elif case == "roulette":
        kw = {"w_th": 0.05, "m": 4.0}
    elif case == "truncated":
        kw = {"flags": 1}
    elif case in ("map", "equal_count"):
        specs, adj = [P.map_source(P.residual_like_map(ph, seed=3))], True
        kw = {"flags": 2} if case == "equal_count" else {}
    got = _run(ph, specs, n, N, adj, tuning, **kw)
    if n > 1024:
        _same(got, _run(ph, specs, n, N, adj, {"live_packets": 1024}, **kw))
    else:   # a pool cannot be smaller: against the whole-grid transport
        _same(got, _run(ph, specs, n, N, adj, noalloc=True, **kw))


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1025])
def test_few_packets(n):
    ph = P.disc_phantom(50, 0.2, 0.02, 8.0, 0.9, seed=3, radius=(1.0, 2.0))
    a = _run(ph, P.four_side_lines(ph), n, 16)
    assert a[1]["packets"] == n and a[1]["launched"] == n
    lost = a[1]["launched"] + a[1]["roulette_gain"] - a[1]["roulette_loss"] - a[1]["absorbed"] - a[1]["escaped"]
    assert abs(lost) < 1e-4 * n
    _same(a, _run(ph, P.four_side_lines(ph), n, 16, tuning={"max_generations": 1, "tile": 5}))


def test_no_power_and_nan_maps():
    """A map of zeros hands no packet to the rounds; one with a NaN gives NaN."""
    from paper_1608_05238_amd import rmc
    ph = P.disc_phantom(50, 0.2, 0.02, 8.0, 0.9, seed=3, radius=(1.0, 2.0))
    med = rmc.Medium.from_phantom(ph)
    q = np.zeros((50, 50))
    co, _ = rmc.mc_adjoint(med, [P.map_source(q)], rmc.make_run(1000, 16))
    assert float(co.abs().max()) == 0.0
    q[3, 4] = np.nan
    co, _ = rmc.mc_adjoint(med, [P.map_source(q)], rmc.make_run(1000, 16))
    assert bool(co.isnan().all())


def test_batch_of_several_problems_in_the_rounds():
    """Lanes of one wave hold packets of different problems."""
    from paper_1608_05238_amd import rmc
    probs = []
    for i, n in enumerate((31, 64, 45)):
        ph = P.disc_phantom(n, 0.25, 0.02 * (i + 1), 6.0, 0.85, seed=i, radius=(0.5, 1.5))
        src = [P.map_source(P.residual_like_map(ph, seed=i))] if i == 1 else P.four_side_lines(ph)
        probs.append(rmc.Problem(rmc.Medium.from_phantom(ph), src, rmc.make_run(3000 * (i + 1), 10, seed=i,
                                                                               stream_tag=i % 2), i == 1))
    a = rmc.mc_run_batch(probs)
    b = rmc.mc_run_batch(probs, tuning={"live_packets": 2048})
    c = rmc.mc_run_batch(probs, tuning={"max_generations": 1})
    for i in range(3):
        assert np.array_equal(a[i][0].cpu().numpy(), b[i][0].cpu().numpy())
        assert np.array_equal(a[i][0].cpu().numpy(), c[i][0].cpu().numpy())
        x, y = rmc.ledger_dict(a[i][1]), rmc.ledger_dict(b[i][1])
        for k in COUNTS:
            assert x[k] == y[k], k
