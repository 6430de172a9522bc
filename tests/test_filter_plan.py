"""Wavefronts per workgroup of the neighbour filter inside clusters (csrc/filter_plan.h, compiled on the host): the span against a simulation of the launch, and the rule at
sets whose workgroups fill the chip once, a little more than once, and many times."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include <chrono>
#include "filter_plan.h"
using namespace nomad_knn;
template <class Fn> double least_us(Fn fn) {
    double least = 1e30;
    for (int i = 0; i < 30; ++i) {
        const auto t0 = std::chrono::steady_clock::now();
        fn();
        least = std::min(least, std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t0).count());
    }
    return least;
}
int main(int argc, char** argv) {   // most, tiles of every group; or 0, slices, candidates, tile, long lists
    if (atoi(argv[1]) == 0) { printf("%d\n", (int)slices_share(atoll(argv[2]), atoll(argv[3]), atoi(argv[4]), atoi(argv[5]))); return 0; }
    std::vector<uint32_t> tstart = {0u};
    for (int a = 2; a < argc; ++a) tstart.push_back(tstart.back() + (uint32_t)atol(argv[a]));
    const std::vector<uint32_t> order = longest_first(tstart);
    std::vector<uint32_t> workgroups;
    for (size_t g = 0; g + 1 < tstart.size(); ++g) workgroups.insert(workgroups.end(), (tstart[g + 1] - tstart[g] + 7) / 8, tstart[g + 1] - tstart[g]);
    const double rule = least_us([&] { volatile int w = filter_waves(tstart, atoi(argv[1])); (void)w; });
    const double sorting = least_us([&] { std::vector<uint32_t> w = workgroups; std::sort(w.begin(), w.end()); volatile uint32_t x = w.empty() ? 0u : w[0]; (void)x; });
    printf("%d %.17g %.17g %g %g\n", filter_waves(tstart, atoi(argv[1])), filter_span(tstart, order, 8), filter_span(tstart, order, atoi(argv[1])), rule, sorting);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("filter_plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(d / "plan.cpp"), "-o", str(d / "plan")],
                   check=True, capture_output=True, text=True)

    def of(most, groups):
        out = subprocess.run([str(d / "plan"), str(most)] + [str(int(c)) for c in groups], check=True, capture_output=True, text=True).stdout.split()
        return (int(out[0]),) + tuple(float(x) for x in out[1:]) if most else int(out[0])
    return of


def _rounds(groups, waves):
    """Workgroups, longest first, each to the unit that is free first: the whole chip's, and an eighth of the work after the other on an eighth of the units."""
    work = [int(c) for c in groups for _ in range(-(-int(c) // waves))]
    before = np.concatenate([[0.0], np.cumsum(work)[:-1]]) / max(1, sum(work))

    def launch(lengths, units):
        at = np.zeros(units)
        for c in sorted(lengths, reverse=True):
            at[at.argmin()] += c
        return at.max()
    return 0.5 * (launch(work, 256) + max(launch([c for c, b in zip(work, before) if int(8 * b) == x], 32) for x in range(8)))


@pytest.mark.parametrize("seed", range(4))
@pytest.mark.parametrize("groups", [20, 70, 250])
def test_the_span_is_a_launch(plan, groups, seed):
    rng = np.random.default_rng(seed)
    for sizes in (np.full(groups, 125), rng.integers(100, 130, groups), np.ceil(rng.gamma(4.0, 25.0, groups))):
        for most in (12, 16):
            _, eight, more = plan(most, sizes)[:3]
            for span, waves in ((eight, 8), (more, most)):
                launch = _rounds(sizes, waves)
                assert 0.70 * launch <= span <= 1.25 * launch            # (the last round is not the mean round)
                if sum(-(-int(c) // waves) for c in sizes) > 1024:       # rounds enough that no single workgroup decides
                    assert 0.90 * launch <= span


def _span(lengths, units):
    lengths = sorted(lengths, reverse=True)
    return max((sum(lengths[:i]) / units + lengths[i] for i in range(0, len(lengths), units)), default=0.0)


@pytest.mark.parametrize("seed", range(4))
@pytest.mark.parametrize("groups", [1, 11, 90, 700])
def test_the_span_by_groups_is_the_one_by_workgroups(plan, groups, seed):
    """Counted by groups; here workgroup by workgroup, with gaps (empty groups), groups of one length, groups that several lists share and long ones among many short ones."""
    rng = np.random.default_rng(seed)
    gaps = rng.integers(0, 60, groups) * (rng.random(groups) < 0.8)
    for sizes in (np.full(groups, 40), gaps, np.ceil(rng.gamma(0.4, 60.0, groups)), np.concatenate([rng.integers(1, 4, groups), [1_500 + 16 * groups]])):
        for most in (12, 16):
            _, eight, more = plan(most, sizes)[:3]
            for span, waves in ((eight, 8), (more, most)):
                work = [int(c) for c in sizes for _ in range(-(-int(c) // waves))]
                total, done, lists = sum(work), 0, [[] for _ in range(8)]
                for c in work:
                    lists[8 * done // total].append(c)
                    done += c
                assert span == pytest.approx(0.5 * (_span(work, 256) + max(_span(l, 32) for l in lists)), rel=1e-12)


def test_the_rule_takes_less_than_sorting_the_workgroups(plan):
    """The device waits for it: a million rows in 256 clusters, 4,000 workgroups, among them one sort of these as the measure."""
    rng = np.random.default_rng(0)
    sizes = rng.gamma(4.0, 1.0, 256)
    waves, _, _, rule, sorting = plan(12, np.ceil(31_250 * sizes / sizes.sum()))
    assert waves == 12 and rule < 0.6 * sorting


def test_the_rule(plan):
    waves = lambda most, groups: plan(most, groups)[0]
    assert waves(8, [125] * 250) == 8                                    # registers for no more
    # clusters of 4,000 rows, tiles of 32: sixteen wavefronts are half as many workgroups
    assert waves(16, [125] * 8) == 8 and waves(16, [125] * 16) == 8      # one round either way
    assert waves(16, [125] * 17) == 16                                   # 272 workgroups, 136
    assert waves(16, [125] * 250) == 16 and waves(12, [125] * 250) == 12
    assert waves(12, [125] * 25) == 8                                    # 400 and 275: two rounds either way
    # rows of 16: twelve are one round of the chip's; eight are hardly more by the chip, but one XCD has two rounds of long ones
    assert waves(12, [-(-n // 16) for n in (5340, 3626, 2814, 2538, 9073, 7306, 1443, 4349, 1129, 2430, 6494)]) == 12
    # as many workgroups of twelve as of eight: a cluster's last one has idle wavefronts
    assert waves(12, [16] * 400) == 8 and waves(12, [16] * 4_000) == 8
    assert waves(16, [17] * 1_000) == 16 and waves(16, [7] * 5_000) == 8
    # one cluster ten times as long as the others decides, however many these are
    assert waves(16, [1_250] + [125] * 10) == 8
    assert waves(16, [1]) == 8 and waves(16, [0, 0]) == 8


def test_which_slices_share(plan):
    share = lambda slices, candidates, tile, long_lists=0: plan(0, [slices, candidates, tile, long_lists]) == 1
    assert share(2, 14_336, 32) and not share(2, 14_335, 32) and not share(1, 10 ** 6, 32)
    assert share(20, 25_600, 32) and not share(20, 25_599, 32)
    assert share(6, 15_360, 16) and not share(6, 15_359, 16)
    assert share(6, 8_192, 32, 1) and not share(6, 8_191, 32, 1) and not share(7, 8_192, 32, 1) and not share(2, 14_335, 16, 1)
    assert share(32, 40_960, 32) and not share(33, 10 ** 6, 32)
