"""Each transport against the FP64 oracle on the same packets: the whole-grid
kernel, the tile kernel's generations and the walk-and-tally rounds, chosen by
the tuning, and the ledger's generations to tell that the chosen one ran.  Bars
as in tests/test_gpu_parity.py."""
import functools

import numpy as np
import pytest

import phantoms as P
from .test_gpu_parity import _assert_maps, _gpu_run, _oracle, _oracle_batches, _rmc

pytestmark = pytest.mark.gpu


def _case(name):
    """phantom, sources, packets, N, run arguments, whether the tally fits one workgroup's LDS"""
    if name == "roulette_grid":
        ph = P.homogeneous(8, 8, 0.5, 2.0, 20.0, 0.0)
        return ph, P.pencil_top_centre(ph), 100_000, 4, dict(seed=23, w_threshold=0.05, roulette_m=4.0), True
    if name == "roulette_disc":
        ph = P.disc_phantom(64, 0.1, 1.0, 12.0, 0.8, seed=14, radius=(0.5, 1.5))
        return ph, P.four_side_lines(ph), 100_000, 16, dict(seed=23, w_threshold=0.05, roulette_m=4.0), False
    if name in ("sin2_fwd", "sin2_adj"):   # p(t) = sin^2(2t) / pi
        ph = P.homogeneous(32, 32, 0.25, 0.05, 8.0, 0.8)
        prof = np.zeros(9)
        prof[0], prof[4] = 1.0, -0.5
        adj = name == "sin2_adj"
        return ph, [P.point_source(4.03, 3.97, prof=prof)], 40_000, 8, dict(seed=17, adjoint=adj, tag=int(adj)), True
    if name == "truncation":
        ph = P.homogeneous(10, 10, 0.5, 1.5, 10.0, 0.3)
        return ph, P.pencil_top_centre(ph), 20_000, 2, dict(w_threshold=0.01, flags=1), True
    if name == "equal_count":
        ph = P.disc_phantom(40, 0.25, 0.03, 6.0, 0.85, seed=6, radius=(1.0, 2.0))
        q = P.residual_like_map(ph, seed=2)
        q[:8, :] = 0.0
        return ph, [P.map_source(q)], 40_000, 8, dict(seed=13, adjoint=True, tag=1, flags=2), False
    # non-scattering and non-absorbing pixels, a g = 1 region
    ph = P.homogeneous(6, 5, 0.4, 0.0, 3.0, 0.5)
    ph.mus[:, 2] = 0.0
    ph.g[3:, :] = 1.0
    ph.mua[1, :] = 0.7
    return ph, [P.point_source(1.0, 1.0)], 5000, 3, dict(seed=11), True


@functools.lru_cache(None)
def _want(name):
    ph, specs, n, N, kw, _ = _case(name)
    return _oracle_batches(_oracle(), ph, specs, n, N, B=8, **kw)


CASES = ["roulette_grid", "roulette_disc", "sin2_fwd", "sin2_adj", "truncation", "equal_count", "edges"]


@pytest.mark.parametrize("case,transport", [(c, t) for c in CASES for t in ("whole_grid", "tiled", "walk")
                                            if t != "whole_grid" or c not in ("roulette_disc", "equal_count")])
def test_transport_against_the_oracle(case, transport):
    ph, specs, n, N, kw, fits = _case(case)
    live = max(1024, n // 5)
    tuning = {"whole_grid": {"grid_max_packets": 1 << 20}, "walk": None,
              # a pool smaller than the run, and generations to (nearly) its end
              "tiled": {"grid_max_packets": 1, "live_packets": live, "finish_packets": 1, "max_generations": 4000}}
    gpu, led = _gpu_run(_rmc(), ph, specs, n, N, tuning=tuning[transport], **kw)
    ora, se = _want(case)
    _assert_maps(f"{case}_{transport}", gpu, ora, se)
    assert led["packets"] == n
    if transport == "whole_grid":
        assert fits and led["generations"] == 0
    elif transport == "tiled":
        assert n // live <= led["generations"] < 4000
    else:
        assert 1 <= led["generations"] <= 64
