"""Where steps of Lloyd's iterations take one launch (csrc/kmeans_plan.h, compiled on the host): both sides of every line."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "kmeans_plan.h"
using namespace nomad_knn;
int main(int argc, char** argv) {   // triples n K d
    for (int a = 1; a + 2 < argc; a += 3) {
        const int64_t n = atoll(argv[a]), K = atoll(argv[a + 1]), d = atoll(argv[a + 2]);
        printf("%d %d %d %d\n", (int)mean_in_one_launch(n, K, d), (int)prepare_in_one_launch(K, d), (int)open_points_are_few(n, K), (int)mean_span(n, K, d));
    }
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("kmeans_plan")
    (d / "plan.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(d / "plan.cpp"), "-o", str(d / "plan")],
                   check=True, capture_output=True, text=True)

    def of(n, K, d_):
        out = subprocess.run([str(d / "plan"), str(n), str(K), str(d_)], check=True, capture_output=True, text=True).stdout.split()
        return [bool(int(x)) for x in out[:3]] + [int(out[3])]
    return of


def test_means(rules):
    assert rules(3_001, 10, 50)[0] and rules(1, 1, 1)[0]
    assert rules(16_384, 64, 64)[0] and not rules(16_385, 64, 64)[0]                  # points
    assert rules(9_090, 10, 64)[0] and not rules(9_091, 10, 64)[0]                    # points and points a cluster
    assert rules(2_857, 2, 64)[0] and not rules(2_858, 2, 64)[0] and rules(1_538, 1, 64)[0] and not rules(1_539, 1, 64)[0]
    assert rules(4_000, 512, 128)[0] and not rules(4_000, 512, 129)[0]                # workgroups
    assert rules(2_048, 1_024, 64)[0] and not rules(2_048, 1_025, 64)[0]
    assert rules(16_384, 512, 64)[0] and not rules(16_384, 513, 64)[0]                # labels read
    assert not rules(16_384, 2_000, 768)[0] and not rules(16_384, 2_147_483_647, 768)[0]


def test_centroids(rules):
    assert rules(5_000, 640, 102)[1] and not rules(5_000, 641, 2)[1]                  # rows
    assert rules(5_000, 85, 768)[1] and not rules(5_000, 86, 768)[1]                  # values


def test_open_points(rules):
    assert rules(16_384, 768, 768)[2] and not rules(16_385, 2, 2)[2] and not rules(16_384, 769, 2)[2]


def test_spans(rules):
    assert [rules(n, 1_000, 255)[3] for n in (98_303, 98_304, 524_287, 524_288)] == [128, 256, 256, 512]      # compute units
    assert [rules(n, 1_000, 256)[3] for n in (65_535, 65_536)] == [128, 256]
    assert [rules(20_736, K, 64)[3] for K in (9, 8, 3, 2)] == [128, 256, 256, 512]                             # partial sums of a cluster
    assert [rules(20_736, K, 768)[3] for K in (5, 4, 1)] == [128, 256, 256] and [rules(300_000, K, 64)[3] for K in (32, 31, 1)] == [256, 512, 512]


PARTS = r"""
#include <stdio.h>
#include <stdlib.h>
#include <string.h>
#include "kmeans_plan.h"
using namespace nomad_knn;
int main(int argc, char** argv) {
    if (!strcmp(argv[1], "refine"))                       // tiles of points
        for (int a = 2; a < argc; ++a) printf("%d\n", (int)refine_tiles(atoll(argv[a])));
    if (!strcmp(argv[1], "counted"))                      // workgroups: those of their wavefronts that count, as list and tile
        for (int g = 0; g < atoi(argv[2]); ++g)
            for (int w = 0; w < 8; ++w)
                if (open_is_counted((uint32_t)g, (uint32_t)w)) printf("%d %d\n", g % 8, g / 8 * 8 + w);
    if (!strcmp(argv[1], "line"))                         // n K d n_tiles steps, rows that are read 16 bytes at a time
        printf("%d\n", (int)products_may_be_alone(atoll(argv[2]), atoll(argv[3]), atoll(argv[4]), atoll(argv[5]), atoll(argv[6]), atoi(argv[7])));
    if (!strcmp(argv[1], "share"))                        // open n K d
        printf("%d\n", (int)products_alone(atoll(argv[2]), atoll(argv[3]), atoll(argv[4]), atoll(argv[5])));
}
"""


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    d = tmp_path_factory.mktemp("kmeans_parts")
    (d / "parts.cpp").write_text(PARTS)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(d / "parts.cpp"), "-o", str(d / "parts")],
                   check=True, capture_output=True, text=True)
    return lambda *a: [int(x) for x in subprocess.run([str(d / "parts")] + [str(x) for x in a], check=True, capture_output=True, text=True).stdout.split()]


def test_what_is_open_is_refined_by_the_whole_chip(ask):
    for tiles in (1, 3, 625, 1_250, 2_048, 4_096, 4_097, 6_251, 9_375, 18_750, 31_250, 1 << 20, 1 << 27):
        t, = ask("refine", tiles)
        assert 1 <= t <= 16                                           # the queue in LDS
        wavefronts = -(-tiles // t)
        assert wavefronts >= min(tiles // 2, 1_024)                   # (four to a workgroup, 256 compute units)


def test_the_sample_of_open_points_is_fair(ask):
    for groups in (128, 131, 256, 300, 1_000, 4_096, 31_250):
        v = ask("counted", groups)
        lists, tiles = v[0::2], v[1::2]
        per_list = [lists.count(x) for x in range(8)]
        share = groups / 64                                           # of a list's groups eight tiles each, one in 64 counted
        assert all(abs(c - share) <= 2 for c in per_list) and min(per_list) >= 1
        if groups == 4_096:                                           # every place among 64 equally often: rows with a period
            assert [sum(t % 64 == p for t in tiles) for p in range(64)] == [8] * 64


def test_large_products_alone(ask):
    line = lambda n, K, d, steps=5, by16=1: ask("line", n, K, d, -(-n // (32 if d <= 256 else 16)), steps, by16) == [1]
    assert line(1_000_000, 256, 128) and line(100_003, 64, 768) and line(50_000, 2_000, 768)
    assert not line(1_000_000, 256, 128, 1)                           # a step that no other follows
    assert not line(1_000_000, 16, 16) and not line(10 ** 9, 4, 8)    # short rows of few centroids
    assert line(524_288, 128, 67, 5, 0) and not line(524_287, 128, 67, 5, 0) and not line(100_003, 128, 231, 5, 0)   # rows that are read word by word
    assert line(131_072, 128, 64) and not line(131_071, 128, 64)      # products
    assert line(32_768, 1_000, 250) and not line(32_736, 1_000, 250)  # workgroups of eight wavefronts
    assert line(16_385, 256, 768) and not line(16_384, 256, 768)      # the open points of few are not refined
    for K, d, part in ((2_000, 768, 16), (256, 128, 32), (128, 64, 128), (64, 768, 16), (64, 257, 22), (64, 256, 64)):
        n = 1 << 20
        assert ask("share", (n - 1) // part, n, K, d) == [1] and ask("share", n // part + 1, n, K, d) == [0]
