"""Which problems take the edge pass that leaves its forces in runs (csrc/edge_plan.h, compiled on the host): the rule's lines, LDS and 16-bit slots."""
import json
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <stdio.h>
#include <stdlib.h>
#include "edge_plan.h"
using namespace nomad;
// argv: n s grouped far pool_size tune_record_sort
int main(int argc, char** argv) {
    if (argc != 7) return 2;
    EdgePlanRequest q;
    q.n = atoll(argv[1]); q.E = 15 * q.n; q.s = atoi(argv[2]); q.grouped = atoi(argv[3]); q.far = atoi(argv[4]);
    q.pool_size = atoi(argv[5]); q.pool_block = q.pool_size ? 4096 : 0; q.tune_record_sort = atoi(argv[6]);
    EdgePlan p = plan_edge_pass(q);
    fit_tiles(p, q, 256, true);
    const RunsPlan x = plan_runs(q, p);
    int split = (uint32_t)x.factor << x.shift == x.points && (int64_t)x.points * x.n_tiles >= q.n && (int64_t)x.points * (x.n_tiles - 1) < q.n;   // and every point in its tile
    const int64_t step = q.n > 3000000 ? 997 : 1;
    for (int64_t i = 0; i < q.n; i += step) split = split && runs_tile_of((uint32_t)i, x.shift, x.magic) == (uint32_t)(i / x.points);
    for (int64_t t = 1; t < x.n_tiles; ++t)
        split = split && runs_tile_of((uint32_t)(t * x.points), x.shift, x.magic) == (uint32_t)t && runs_tile_of((uint32_t)(t * x.points - 1), x.shift, x.magic) == (uint32_t)(t - 1);
    printf("{\"use\": %d, \"sums\": %d, \"tiles\": %u, \"points\": %u, \"split\": %d, \"slots\": %zu, \"edges\": %d, \"lds\": %zu, \"sums_lds\": %zu, \"max_lds\": %zu}\n",
           (int)x.use, x.sums_lanes, x.n_tiles, x.points, split, runs_slots(q.s), runs_block_edges(q.s), runs_lds_bytes(q.s, x.n_tiles),
           (size_t)16 * x.points + (size_t)(kBinBlock / 64) * tile_sums_queue(x.sums_lanes) * 8, kMaxLdsBytes);
    return 0;
}
"""


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("runs_plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)

    def plan(n, s=5, grouped=0, far=0, pool=0, sort=0):
        out = subprocess.run([str(exe)] + [str(int(v)) for v in (n, s, grouped, far, pool, sort)], check=True, capture_output=True, text=True)
        return json.loads(out.stdout)
    return plan


def test_tiles_fill_the_compute_units(planner):
    assert [planner(n)["tiles"] for n in (100_000, 300_000, 600_000, 900_000)] == [256, 256, 256, 220]
    assert [planner(n, s=2, grouped=1)["tiles"] for n in (3_000_000, 6_000_011)] == [510, 733]   # 184 x 32 points; 8,192


def test_the_lines(planner):
    assert [planner(n)["use"] for n in (2, 100_000, 900_000)] == [1, 1, 1]
    assert planner(100_000, s=9)["use"] == 0 and planner(100_000, pool=1024)["use"] == 0 and planner(100_000, sort=1)["use"] == 0
    assert planner(6_000_000, s=2, grouped=1)["use"] == 1
    assert [planner(n, grouped=1, far=1)["use"] for n in (256 * 8192, 256 * 8192 + 1)] == [1, 0]
    assert planner(60_000_000, s=2, grouped=1)["use"] == 0           # records that are not sorted


@pytest.mark.parametrize("s", range(9))
def test_slots_and_lds(planner, s):
    for n in (2, 257, 5_000, 40_961, 99_999, 300_000, 600_001, 1_400_000, 2_000_000, 2_200_000, 8_000_000, 30_000_000):
        p = planner(n, s=s, grouped=1)
        assert p["slots"] % 64 == 0 and p["slots"] >= p["edges"] * (s + 1) + p["edges"] // 32 and p["slots"] < 65_536
        assert p["edges"] % 64 == 0
        if p["use"]:
            assert p["points"] <= 8192 and p["tiles"] < 65_536 and p["split"]
            assert 2 * p["lds"] <= p["max_lds"] and p["sums_lds"] <= p["max_lds"] and p["sums"] in (8, 16, 32)
