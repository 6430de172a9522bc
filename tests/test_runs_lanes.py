"""Lanes of a segment of k_tile_sums that plan_runs gives the problems of tests/test_gpu_runs_told.py: each of the three kernels runs there.  Sparse graphs: the rule's lines."""
import os
import subprocess

import pytest

from tests.test_gpu_runs_told import LANES
from tests.test_runs_plan import planner  # noqa: F401


def test_lanes(planner):  # noqa: F811
    assert {planner(n, s=s)["sums"] for n, s, _, _ in LANES} == {8, 16, 32}
    for n, s, _, lanes in LANES:
        p = planner(n, s=s)
        assert p["use"] == 1 and p["sums"] == lanes, (n, s)


DRIVER = r"""
#include <stdio.h>
#include <stdlib.h>
#include "edge_plan.h"
using namespace nomad;
int main(int argc, char** argv) {   // triples n, E, s
    for (int i = 1; i + 2 < argc; i += 3) {
        EdgePlanRequest q;
        q.n = atoll(argv[i]); q.E = atoll(argv[i + 1]); q.s = atoi(argv[i + 2]);
        EdgePlan p = plan_edge_pass(q);
        fit_tiles(p, q, 256, true);
        printf("%d", (int)plan_runs(q, p).use);
    }
    return 0;
}
"""


@pytest.mark.parametrize("n,E,s", [(10_225, 8_192, 5), (10_225, 32_768, 2), (10_225, 32_768, 1), (10_225, 8_192, 0), (131_071, 8_192, 6), (131_072, 16_384, 3), (524_287, 16_384, 4), (524_288, 32_768, 5),
                                   (2_000_000, 32_768, 0)])
def test_sparse(tmp_path, n, E, s):
    (tmp_path / "plan.cpp").write_text(DRIVER)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    subprocess.run(["g++", "-std=c++17", "-I", os.path.join(root, "paper_2505_15511_amd", "csrc"), str(tmp_path / "plan.cpp"), "-o", str(tmp_path / "plan")], check=True)
    asked = [(n, E, s), (n, E + 1, s), (n, 1, s), (10_224, E, s), (n, E, 7)]          # at the line, beyond it; embeddings whose sums fit LDS, and blocks of 512, always
    got = subprocess.run([str(tmp_path / "plan")] + [str(v) for a in asked for v in a], check=True, capture_output=True, text=True).stdout
    assert got == "01011"
