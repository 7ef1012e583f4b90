"""Small grids on both sides of the packet count up to which they walk, and of
the one from which they are tiled: the same maps bit for bit, and the same
event counts, as the whole-grid transport of mc_run_noalloc."""
import pytest

import phantoms as P
from .test_gpu_walk import _run, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1 << 17, (1 << 17) + 1, 200_000])
@pytest.mark.parametrize("adjoint", [False, True])
def test_small_grids_on_both_sides_of_the_rule(n, adjoint):
    ph = P.disc_phantom(14, 0.4, 0.3, 6.0, 0.8, seed=2, radius=(1.0, 2.0))
    specs = [P.map_source(P.residual_like_map(ph, seed=2))] if adjoint else P.four_side_lines(ph)
    want = _run(ph, specs, n, 5, adjoint, noalloc=True)
    _same(_run(ph, specs, n, 5, adjoint), want)
    _same(_run(ph, specs, n, 5, adjoint, {"grid_max_packets": 1000}), want)
