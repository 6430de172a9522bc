"""Lanes of a segment of k_tile_sums that plan_runs gives the problems of tests/test_gpu_runs_told.py: each of the three kernels runs there."""
from tests.test_gpu_runs_told import LANES
from tests.test_runs_plan import planner  # noqa: F401


def test_lanes(planner):  # noqa: F811
    assert {planner(n, s=s)["sums"] for n, s, _, _ in LANES} == {8, 16, 32}
    for n, s, _, lanes in LANES:
        p = planner(n, s=s)
        assert p["use"] == 1 and p["sums"] == lanes, (n, s)
