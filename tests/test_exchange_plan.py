"""Which problems take the exchanged edge pass and with what shapes (csrc/edge_plan.h, compiled on the host): the rule's line, the LDS
of its four kernels, 16-bit slots, and the knobs that keep a problem on the sorted pass."""
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
// argv: n E s pool_size tune_exchange tune_record_sort [batches]
int main(int argc, char** argv) {
    if (argc != 7 && argc != 8) return 2;
    EdgePlanRequest q;
    q.n = atoll(argv[1]); q.E = atoll(argv[2]); q.s = atoi(argv[3]); q.pool_size = atoi(argv[4]); q.pool_block = q.pool_size ? 4096 : 0;
    q.tune_exchange = atoi(argv[5]); q.tune_record_sort = atoi(argv[6]);
    if (argc == 8) q.batches = atoi(argv[7]);
    EdgePlan p = plan_edge_pass(q);
    fit_tiles(p, q, 256, true);
    const ExchangePlan x = plan_exchange(q, p);
    printf("{\"use\": %d, \"pairs\": %d, \"rows\": %d, \"sums\": %d, \"parts\": %u, \"tiles\": %u, \"tile_bits\": %d, \"slots\": %zu, \"edges\": %d, "
           "\"deal_lds\": %zu, \"rows_lds\": %zu, \"edges_lds\": %zu, \"sums_lds\": %zu, \"max_lds\": %zu}\n",
           (int)x.use, (int)x.pairs, x.rows_lanes, x.sums_lanes, x.parts, p.n_bins, p.tile_bits, exchange_slots(q.s), exchange_block_edges(q.s),
           exchange_deal_lds_bytes(q.s, p.n_bins), exchange_rows_lds_bytes(x), exchange_edges_lds_bytes(q.s), tile_sums_lds_bytes(x), kMaxLdsBytes);
    return 0;
}
"""


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    d = tmp_path_factory.mktemp("exchange_plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)

    def plan(n, s=5, E=None, pool=0, exchange=0, sort=0, batches=1):
        out = subprocess.run([str(exe)] + [str(int(v)) for v in (n, 15 * n if E is None else E, s, pool, exchange, sort, batches)], check=True, capture_output=True, text=True)
        return json.loads(out.stdout)
    return plan


def test_the_line(planner):
    assert [planner(n)["use"] for n in (2_000, 999_999, 1_000_000, 10_000_000)] == [0, 0, 1, 1]
    assert [planner(n, s=2)["use"] for n in (1_499_999, 1_500_000)] == [0, 1]
    assert planner(10_000_000, pool=1024)["use"] == 0 and planner(10_000_000, s=0)["use"] == 0 and planner(10_000_000, s=9)["use"] == 0
    assert planner(10_000_000, E=0)["use"] == 0
    assert planner(60_000_000, s=2)["use"] == 0                      # runs shorter than two references
    assert planner(10_000_000, sort=1)["use"] == 0 and planner(10_000_000, exchange=2)["use"] == 0
    assert planner(2_000, exchange=1)["use"] == 1 and planner(10_000_000, exchange=1, sort=1)["use"] == 1


@pytest.mark.parametrize("s", range(1, 9))
def test_short_sub_steps_stay_on_the_sorted_pass(planner, s):
    n, E = 4_000_000, 60_000_000
    most = E * (s + 1) // 8_000_000                                  # sub-steps of eight million references
    assert planner(n, s, E, batches=1)["use"] == planner(n, s, E, batches=most)["use"] == 1
    assert planner(n, s, E, batches=most + 1)["use"] == 0
    assert planner(n, s, 3_000_000, batches=1)["use"] == 1 and planner(n, s, E, exchange=1, batches=10_000)["use"] == 1


@pytest.mark.parametrize("s", range(1, 9))
def test_shapes_fit(planner, s):
    for n in (2, 300, 70_000, 1_000_000, 2_097_152, 2_097_153, 5_000_000, 10_000_000, 20_000_000):
        p = planner(n, s, exchange=1)
        assert p["use"] == 1
        assert p["edges"] % 64 == 0 and p["slots"] >= p["edges"] * (s + 1) + 2 * (p["edges"] // 64) and p["slots"] % 64 == 0
        assert p["slots"] < 65_536                                   # slots and run lengths are 16-bit
        assert p["tile_bits"] + p["pairs"] <= 16                     # so is what a tile knows of a point
        assert 2 * p["edges_lds"] <= 160 * 1024
        assert max(p["deal_lds"], p["rows_lds"], p["sums_lds"]) <= p["max_lds"]
        assert 1 <= p["parts"] <= 1024


SMALL = r"""
#include <stdio.h>
#include <stdlib.h>
#include "edge_plan.h"
using namespace nomad;
int main(int argc, char** argv) {
    EdgePlanRequest q;
    q.n = atoll(argv[1]); q.E = atoll(argv[2]); q.s = atoi(argv[3]); q.pool_size = atoi(argv[4]); q.pool_block = q.pool_size ? 4096 : 0; q.tune_phases = atoi(argv[5]); q.far = argc > 6 && atoi(argv[6]);
    EdgePlan p = plan_edge_pass(q);
    fit_tiles(p, q, 256, true);
    printf("%d %zu %zu\n", plan_small(q, p, 256), small_lds_bytes(q.n), kMaxLdsBytes);
    return 0;
}
"""


def test_sums_in_lds(tmp_path):
    """Embeddings whose sums fit a workgroup's LDS, the workgroups they get, and what keeps them on the other passes."""
    (tmp_path / "small.cpp").write_text(SMALL)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(tmp_path / "small.cpp"), "-o",
                    str(tmp_path / "small")], check=True, capture_output=True, text=True)

    def plan(n, E, s=5, pool=0, phases=0, far=0):
        wg, lds, most = map(int, subprocess.run([str(tmp_path / "small")] + [str(v) for v in (n, E, s, pool, phases, far)], check=True, capture_output=True,
                                                text=True).stdout.split())
        assert wg == 0 or lds <= most
        return wg
    assert plan(2_000, 46_734) == 46 and plan(1, 1) == 1 and plan(2, 10 ** 7) == 256
    assert plan(10_224, 300_000) > 0 and plan(10_225, 300_000) == 0
    for n in (5_000, 8_000, 10_224):
        assert plan(n, 10 ** 6) * 16 * n <= 12 << 20
    assert plan(2_000, 46_734, s=9) == plan(2_000, 46_734, pool=1024) == plan(2_000, 46_734, phases=2) == plan(2_000, 0) == 0
    # one round more than there is room for: all do two, with half the sums
    assert plan(10_200, 77 * 1024) == 77 and plan(10_200, 77 * 1024 + 1) == 39 and plan(10_200, 3 * 77 * 1024) == 77 and plan(2_000, 300 * 1024) == 256
    # sampled far field: records where a workgroup had too many rounds
    for n, s, records, lds in ((8_000, 2, 20 * 8_000, 250 * 8_000), (8_000, 8, 45 * 8_000, 60 * 8_000), (9_000, 8, 4 * 9_000, 12 * 9_000), (10_200, 5, 4 * 10_200, 45 * 10_200)):
        assert plan(n, records, s, far=1) > 0 and plan(n, lds, s, far=1) == 0 and plan(n, lds, s) > 0
    assert all(plan(5_242, k * 5_242, s, far=1) > 0 for k in (1, 30, 500) for s in range(9))
    # no negatives
    assert plan(9_000, 4 * 9_000, 0) > 0 and plan(9_000, 8 * 9_000, 0) == 0 and plan(9_000, 12 * 9_000, 0) == 0 and plan(9_000, 30 * 9_000, 0) > 0
    assert plan(7_000, 12 * 7_000, 0) == 0 and plan(7_000, 20 * 7_000, 0) > 0 and plan(5_000, 20 * 5_000, 0) > 0
