"""grid_max_packets chooses the kernel of a run on a small grid: up to that
many packets the whole-grid kernel (no generations), also where such a run
would walk by default.  The default value passed on, as a dict of all
defaults holds it, is no choice.  The maps are the same bits."""
import pytest

import phantoms as P
from .test_gpu_walk import _run, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 20_000, 1 << 17])
def test_the_caller_chooses(n):
    from paper_1608_05238_amd import rmc
    ph = P.disc_phantom(14, 0.4, 0.3, 6.0, 0.8, seed=2, radius=(1.0, 2.0))
    specs = P.four_side_lines(ph)
    walk = _run(ph, specs, n, 5)
    assert walk[1]["generations"] >= 1
    for tuning in ({"grid_max_packets": n}, {"grid_max_packets": 1 << 20}):
        grid = _run(ph, specs, n, 5, tuning=tuning)
        assert grid[1]["generations"] == 0, tuning
        _same(grid, walk)
    same = _run(ph, specs, n, 5, tuning=rmc.default_tuning())
    assert same[1]["generations"] == walk[1]["generations"]
    if n > 1:
        other = _run(ph, specs, n, 5, tuning={"grid_max_packets": n - 1})
        assert other[1]["generations"] >= 1
        _same(other, walk)
