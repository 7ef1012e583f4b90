"""The tile kernel's schedule -- when it looks after its lanes, pauses packets,
shares out the records held ahead at a job's end -- against the walk-and-tally
rounds on the same packets, over the knobs that bring out its edges: bitwise
equal maps and equal event counts (the sums are of integers, so no order of
arrival may show).  A pool smaller than the run makes the generations launch
and move the packets; finish_packets 1 makes them move nearly all to the end."""
import numpy as np
import pytest

import phantoms as P
from .test_gpu_walk import _run, _same

pytestmark = pytest.mark.gpu

BASE = {"finish_packets": 1, "max_generations": 4000}


@pytest.mark.parametrize("knobs", [
    {"live_packets": 9000},                                              # jobs of several packets a lane
    {"live_packets": 9000, "tile": 50},                                  # one tile: the grid's edge is the tile's
    {"live_packets": 9000, "job_packets": 64, "min_job_packets": 64},    # jobs of less than a packet a lane
    {"live_packets": 5000, "max_visits": 1},                             # every visit pauses
    {"live_packets": 5000, "max_visits": 3, "tail_visits": 1, "quiet_percent": 100},   # quiet from the first look
    {"live_packets": 5000, "tail_visits": 1000, "quiet_percent": 1},     # stays run to their end
    {"live_packets": 5000, "tile": 2},                                   # stays of a few segments
    {"live_packets": 1100, "tile": 7, "flush_track": 0.3},               # visits flushed in parts
])
@pytest.mark.parametrize("n_harm", [1, 16, 32])
def test_tile_schedule_does_not_show(knobs, n_harm):
    ph = P.disc_phantom(25, 0.4, 0.02, 8.0, 0.9, seed=3, radius=(1.0, 2.0))
    specs = P.four_side_lines(ph)
    n = 10_000
    kw = {"w_th": 0.02, "m": 5.0}   # roulette deaths too
    if "flush_track" in knobs:   # in parts also in the rounds: the parts' roundings are of the result
        want = _run(ph, specs, n, n_harm, tuning={"flush_track": knobs["flush_track"]}, **kw)
    else:
        want = _run(ph, specs, n, n_harm, **kw)
    _same(_run(ph, specs, n, n_harm, tuning={**BASE, **knobs}, **kw), want)


@pytest.mark.parametrize("n", [1025, 1087, 2049])
def test_a_job_of_a_few_more_packets_than_lanes(n):
    """Some lanes hold a record ahead when the job has no more: free ones take it."""
    ph = P.homogeneous(12, 12, 0.3, 0.05, 6.0, 0.8)
    specs = [P.point_source(1.9, 2.0)]
    _same(_run(ph, specs, n, 4, tuning={**BASE, "live_packets": 1024}), _run(ph, specs, n, 4))
    _same(_run(ph, specs, n, 4, tuning={**BASE, "live_packets": n - 1}), _run(ph, specs, n, 4))
