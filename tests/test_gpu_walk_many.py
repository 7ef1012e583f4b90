"""Runs of so many packets that a walking wave works out its own random
numbers, and one packet fewer, against the generations of the tile kernel:
bitwise equal maps and equal event counts.  (live_packets 2^16 makes the
generations launch the packets; finish_packets 1 makes them move nearly all.)"""
import numpy as np
import pytest

import phantoms as P
from .test_gpu_walk import COUNTS, _run, _same

pytestmark = pytest.mark.gpu

MANY = 1 << 19   # the rule's line: twice the lanes that walk at once


@pytest.mark.parametrize("n", [MANY - 1, MANY, MANY + 65])
@pytest.mark.parametrize("case", ["disc", "map"])
def test_many_packets_equal_generations(n, case):
    ph = P.disc_phantom(40, 0.25, 0.3, 6.0, 0.8, seed=3, radius=(1.0, 2.0))
    adj = case == "map"
    specs = [P.map_source(P.residual_like_map(ph, seed=3))] if adj else P.four_side_lines(ph)
    kw = {"w_th": 0.05, "m": 4.0}
    got = _run(ph, specs, n, 8, adj, **kw)
    _same(got, _run(ph, specs, n, 8, adj, {"live_packets": 1 << 16, "finish_packets": 1, "max_generations": 4000}, **kw))


def test_many_packets_of_two_problems():
    """Lanes change from one problem's packets to the other's."""
    from paper_1608_05238_amd import rmc
    probs = []
    for i, n in enumerate((33, 40)):
        ph = P.disc_phantom(n, 0.25, 0.4 * (i + 1), 6.0, 0.85, seed=i, radius=(0.5, 1.5))
        probs.append(rmc.Problem(rmc.Medium.from_phantom(ph), P.four_side_lines(ph),
                                 rmc.make_run(MANY // 2 + 100 * i, 5, seed=i), False))
    a = rmc.mc_run_batch(probs)
    b = rmc.mc_run_batch(probs, tuning={"live_packets": 1 << 16, "finish_packets": 1, "max_generations": 4000})
    for i in range(2):
        assert np.array_equal(a[i][0].cpu().numpy(), b[i][0].cpu().numpy())
        x, y = rmc.ledger_dict(a[i][1]), rmc.ledger_dict(b[i][1])
        for k in COUNTS:
            assert x[k] == y[k], k
