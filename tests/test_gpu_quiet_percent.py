"""quiet_percent is the percentage that the caller gives, in jobs of any size.
One job of 8999 packets (more than eight a thread), which pause for this rule
alone (no limit of visits): at 77 percent of its 1024 threads at most 788 stays
are left to pause, fewer than the 800 at which the generations end, so the
first one is the last."""
import pytest

import phantoms as P
from .test_gpu_walk import _run, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("percent", [10, 56, 77])
def test_percentage_as_given(percent):
    ph = P.homogeneous(20, 20, 0.3, 0.01, 3.0, 0.8)
    specs, n = [P.point_source(3.1, 3.0)], 9000
    one_job = {"live_packets": n - 1, "grid_max_packets": 1, "job_packets": 32768, "min_job_packets": 16384,
               "finish_packets": 100, "max_generations": 2000, "max_visits": 1 << 30}
    got = _run(ph, specs, n, 16, tuning={**one_job, "quiet_percent": percent})
    assert got[1]["generations"] == 1
    _same(got, _run(ph, specs, n, 16))
