"""The transport that bench.py names for a run on a small grid, against the
rule in the kernel source."""
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_walk_limit_is_the_library_s():
    import bench
    with open(os.path.join(ROOT, "paper_1608_05238_amd", "csrc", "mcrad.hip")) as f:
        a, b = re.search(r"kDirectMax = (\d+)ull << (\d+);", f.read()).groups()
    assert bench.WALK_MAX == int(a) << int(b)


@pytest.mark.parametrize("n,generations,mode", [(100_000, 2, "walk and tally"), (1_000_000, 0, "whole grid"),
                                                (3 << 19, 3, "walk and tally"), ((3 << 19) + 1, 36, "tiled"),
                                                (2_000_000, 0, "whole grid"), (100_000_000, 36, "tiled")])
def test_mode(n, generations, mode):
    import bench
    assert bench.transport_mode(n, generations) == mode
