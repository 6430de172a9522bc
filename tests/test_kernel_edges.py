"""Sizes at which the index, initialisation and quality kernels change their shape: the ends of tiles, of list and dimension
classes, of the parallel sums; against the oracles."""
import numpy as np
import pytest
import torch

from oracle import kmeans_oracle as km
from oracle import knn_oracle as ko
from oracle import metrics_oracle as mo
from oracle import pca_oracle as po
from paper_2505_15511_amd import kmeans_lloyd, kmeans_lsh_init, knn_in_clusters, neighbourhood_preservation, pca_init, pipeline


@pytest.mark.parametrize("n,m,seed", [(16, 2, 0), (1000, 125, 3), (80001, 10000, 7), (999, 500, 1), (5000, 5, 2**40 + 9), (1000, 0, 4)])
def test_sampled_queries_are_the_head_of_the_permutation(n, m, seed):
    ref = torch.randperm(n, generator=torch.Generator().manual_seed(seed))[:m]
    assert torch.equal(pipeline.sample_without_replacement(n, m, seed), ref)


def test_long_permutations_are_torch_s_own(monkeypatch):
    asked = []
    monkeypatch.setattr(pipeline.torch, "randperm", lambda n, generator: asked.append(n) or torch.arange(5))
    for n in (214_748_363, 214_748_364, 214_748_370, 1 << 31):      # 32-bit draws up to (2^32 - 1) / 20 entries
        pipeline.sample_without_replacement(n, 4, 1)
    assert asked == [214_748_364, 214_748_370, 1 << 31]


@pytest.mark.gpu
@pytest.mark.parametrize("d", [16, 17, 128, 129, 256, 257, 384, 385])
@pytest.mark.parametrize("k", [1, 8, 9, 16, 17, 32])
def test_filter_classes(d, k):
    rng = np.random.default_rng(d * 100 + k)
    c = rng.permutation(np.repeat(np.arange(6), [31, 33, 64, 1, 290, 129]))
    X = (rng.normal(size=(len(c), d)) + 3.0 * rng.normal(size=(6, d))[c]).astype(np.float32)
    assert np.array_equal(knn_in_clusters(X, c, 6, k).astype(np.int64), ko.in_cluster_knn(X, c, k)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,k", [(32 * 1024 + 5, 9, 15), (16 * 1024 + 5, 260, 15), (16 * 1024 + 5, 140, 20)])
def test_filter_with_the_wide_workgroup(n, d, k):
    rng = np.random.default_rng(n)
    c = rng.integers(0, 60, n)
    X = rng.normal(size=(n, d)).astype(np.float32)
    out = knn_in_clusters(torch.from_numpy(X).cuda(), torch.from_numpy(c).cuda(), 60, k).cpu().numpy()
    assert np.array_equal(out.astype(np.int64), ko.in_cluster_knn(X, c, k)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("n,k,layout", [(1023, 15, "normal"), (1024, 15, "normal"), (1500, 32, "normal"), (3000, 1, "grid"), (3000, 15, "grid"),
                                        (2500, 15, "outliers"), (2500, 15, "line"), (2000, 32, "point")])
def test_plane_neighbours(n, k, layout):
    rng = np.random.default_rng(n + k)
    Y = rng.normal(size=(n, 2)).astype(np.float32)
    if layout == "grid":
        Y = rng.integers(0, 12, size=(n, 2)).astype(np.float32)          # ties and duplicates in bulk
    elif layout == "outliers":
        Y[:3] = [[1e6, 1e6], [-1e6, 1e6], [1e6, -3e5]]                   # nearly all points in one cell
    elif layout == "line":
        Y[:, 1] = 0.25
    elif layout == "point":
        Y[:] = 1.5
        Y[-5:] += 1.0
    X = np.concatenate([Y, 0.3 * rng.normal(size=(n, 3)).astype(np.float32)], axis=1)
    q = rng.permutation(n)[:200].astype(np.int32)
    q[:3] = [0, n - 1, n - 2]
    q = np.unique(q).astype(np.int32)
    assert neighbourhood_preservation(X, Y, k, q)[0] == mo.neighbourhood_preservation(X, Y, k, q)[0]


@pytest.mark.gpu
@pytest.mark.parametrize("n,d,K", [(513, 64, 4), (1024, 65, 8), (1537, 66, 1), (2000, 128, 15), (2000, 130, 2), (1300, 132, 10), (1300, 260, 3), (127, 6, 1)])
def test_centroids_of_large_clusters(n, d, K):
    rng = np.random.default_rng(n + d)
    X = (rng.normal(size=(n, d)) * 10.0 ** rng.integers(-6, 4, size=(1, d))).astype(np.float32)
    C0 = X[rng.choice(n, K, replace=False)].copy()
    C_ref, lab_ref, it_ref, _ = km.lloyd(X, C0, 4)
    C, lab, it, _ = kmeans_lloyd(X, C0, 4)
    assert it == it_ref and np.array_equal(lab.astype(np.int64), lab_ref) and np.array_equal(C, C_ref)


@pytest.mark.gpu
@pytest.mark.parametrize("n", [128, 1024, 1026, 5000])
def test_means_on_a_rounding_boundary_are_added_in_order(n):
    rng = np.random.default_rng(n)
    X = np.full((n, 4), 1.0, np.float32)
    half = rng.permutation(n)[:n // 2]
    X[half, 0] = np.float32(1.0 + 2.0**-23)          # the mean lies half way between two float32 values
    X[:, 1] = rng.normal(size=n)
    X[half, 2] = -1.0                                # the sum is zero exactly
    X[half[0], 3] = np.inf
    C_ref = km.update(X, np.zeros(n, np.int64), X[:1])
    C, _ = kmeans_lsh_init(X, 1, np.array([[0.0, 1.0, 0.0, 0.0]], np.float32), np.array([3], np.int32), return_buckets=True)
    assert np.array_equal(C, C_ref)


@pytest.mark.gpu
@pytest.mark.parametrize("b", [8, 9, 16, 17, 30])
@pytest.mark.parametrize("n,d", [(255, 15), (257, 16), (600, 33)])
def test_hash_planes(n, d, b):
    rng = np.random.default_rng(n + b)
    X = rng.normal(size=(n, d)).astype(np.float32)
    planes, anchors = rng.normal(size=(b, d)).astype(np.float32), rng.choice(n, b).astype(np.int32)   # anchors lie on their plane
    X[n // 2:n // 2 + 20] = X[anchors[rng.integers(0, b, 20)]]
    C_ref, b_ref = km.lsh_init(X, planes, anchors, 50)
    C, buckets = kmeans_lsh_init(X, 50, planes, anchors, return_buckets=True)
    assert np.array_equal(buckets.astype(np.int64), b_ref) and np.array_equal(C, C_ref)


@pytest.mark.gpu
@pytest.mark.parametrize("n,d", [(70, 3), (500, 9), (1000, 127), (1000, 128), (1000, 129), (900, 257)])
def test_principal_axes(n, d):
    rng = np.random.default_rng(d)
    X = (rng.normal(size=(n, d)) * np.r_[9.0, 5.0, np.ones(d - 2)] + rng.normal(size=d)).astype(np.float32)
    ref, lam_ref = po.pca_init(X, 0.0)
    theta, st = pca_init(X, 0.0, return_stats=True)
    assert np.allclose(st["eigenvalues"], lam_ref, rtol=1e-10) and st["residual"] <= 1e-9
    assert np.abs(theta - ref).max() <= 1e-5 * np.abs(ref).max()


# ---------------------------------------------------------------- the edge pass
def test_fitted_tiles(tmp_path):
    import json
    import os
    import subprocess
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src = tmp_path / "plan.cpp"
    src.write_text(r'''
#include <stdio.h>
#include <stdlib.h>
#include "edge_plan.h"
using namespace nomad;
int main(int, char** argv) {
    EdgePlanRequest q;
    q.n = atoll(argv[1]); q.E = 30 * q.n; q.s = atoi(argv[2]); q.pool_size = atoi(argv[3]); q.pool_block = 8192; q.pool_line = 16; q.pool_distinct = true;
    EdgePlan p = plan_edge_pass(q);
    const uint32_t before = p.n_bins;
    fit_tiles(p, q, 256);
    printf("[%d, %u, %u, %d, %d, %d, %d, %d]\n", p.tile_bits, p.n_bins, before, (int)p.sorted, p.pool_rounds, p.flush_rounds, p.bin_block,
           (int)edge_tables_fit(p, q));
}
''')
    exe = str(tmp_path / "plan")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(root, "paper_2505_15511_amd", "csrc"), str(src), "-o", exe], check=True)
    for n, s, pool in [(1, 5, 0), (17, 5, 0), (2_000, 5, 0), (2_184, 8, 0), (2_185, 8, 0), (4_097, 2, 0), (3_001, 5, 4096), (65_535, 5, 0), (65_536, 5, 0), (65_793, 8, 0), (1_000_000, 5, 0), (2_097_152, 2, 0), (2_097_153, 8, 0),
                       (10_000_000, 5, 0), (10_000_000, 2, 0), (60_000_000, 2, 0), (3_000_017, 5, 4096)]:
        bits, bins, before, is_sorted, pool_rounds, rounds, block, fits = json.loads(subprocess.run([exe, str(n), str(s), str(pool)], check=True, capture_output=True, text=True).stdout)
        assert (bins - 1) << bits < n <= bins << bits and fits
        assert bins <= max(before, 256) and bits >= 4
        if is_sorted and not pool_rounds:
            assert (n >> bits) <= 256 or bits == 13
            assert rounds in (1, 2) and (block == 256) == (30 * n <= 256 * 256)
        elif n > 65_536:
            assert bins == before


@pytest.mark.gpu
@pytest.mark.parametrize("n", [255, 257, 4_097, 7_000, 65_537, 140_001])
@pytest.mark.parametrize("s", [0, 1, 5, 7, 8])
@pytest.mark.parametrize("grouped", [False, True])
def test_sorted_records_reach_their_points(n, s, grouped):
    """The binned path against fixed-point atomics: the same sums of the same forces, head sums in another order."""
    from paper_2505_15511_amd import PATH_BINNED, PATH_FIXED_ATOMICS, Nomad, workloads
    R = 9
    g = workloads.planted_knn_graph(n, R, 6, 0.05, 11 + s, device="cuda")
    groups = torch.arange(R, dtype=torch.int32, device="cuda") if grouped else None
    theta = 0.1 * torch.randn(n, 2, generator=torch.Generator().manual_seed(n))
    grads = []
    for tune in (None, PATH_FIXED_ATOMICS):
        nm = Nomad(n, R, s, 5.0, 10, 1.0, 3, tune={"scatter_path": tune} if tune else {})
        nm.set_graph(g["row_ptr"], g["col_idx"], None, g["cluster_of"], groups)
        assert nm.scatter_path() == (tune or PATH_BINNED)
        nm.set_embedding(theta)
        nm.epoch(0)
        nm.set_embedding(theta)
        nm.epoch(1)
        grads.append(np.asarray(nm.get_gradient(), dtype=np.float64))
    assert np.abs(grads[0] - grads[1]).max() <= 1e-6 * np.abs(grads[1]).max()


# ---------------------------------------------------------------- rows whose filter keys are not finite
@pytest.mark.gpu
@pytest.mark.parametrize("d,k", [(20, 8), (260, 15), (140, 20)])
@pytest.mark.parametrize("outlier", [2e18, 1e20, 3e38])
def test_neighbours_next_to_a_sentinel(d, k, outlier):
    rng = np.random.default_rng(d)
    c = rng.permutation(np.repeat(np.arange(4), [12, 200, 90, 1]))
    X = (rng.normal(size=(len(c), d)) + 3.0 * rng.normal(size=(4, d))[c]).astype(np.float32)
    X[np.flatnonzero(c == 0)[0], 3] = outlier
    X[np.flatnonzero(c == 1)[:2], 0] = [outlier, -outlier]
    out, stats = knn_in_clusters(X, c, 4, k, return_stats=True)
    assert np.array_equal(out.astype(np.int64), ko.in_cluster_knn(X, c, k)[0])
    assert outlier < 1e19 or stats["fallback_queries"] >= 212


@pytest.mark.gpu
@pytest.mark.parametrize("d,K", [(20, 7), (260, 40), (400, 3)])
@pytest.mark.parametrize("outlier", [1e20, -3e38])
def test_partition_next_to_a_sentinel(d, K, outlier):
    rng = np.random.default_rng(d + K)
    X = rng.normal(size=(1200, d)).astype(np.float32)
    X[7, 2] = outlier
    C0 = X[rng.choice(1200, K, replace=False)].copy()
    C_ref, lab_ref, it_ref, _ = km.lloyd(X, C0, 3)
    C, lab, it, _ = kmeans_lloyd(X, C0, 3)
    assert it == it_ref and np.array_equal(lab.astype(np.int64), lab_ref) and np.array_equal(C, C_ref)


@pytest.mark.gpu
def test_partition_far_from_its_starting_centroids():
    X = (1e-15 * np.random.default_rng(1).normal(size=(1200, 16))).astype(np.float32)   # the points' scale times the centroids' norms overflows
    C0 = np.stack([X[0], X[1] + np.float32(3e17), X[2] - np.float32(1e17)]).astype(np.float32)
    C_ref, lab_ref, it_ref, _ = km.lloyd(X, C0, 3)
    C, lab, it, _ = kmeans_lloyd(X, C0, 3)
    assert it == it_ref and np.array_equal(lab.astype(np.int64), lab_ref) and np.array_equal(C, C_ref)


@pytest.mark.gpu
@pytest.mark.parametrize("value", [np.nan, np.inf])
def test_labels_stay_in_range_whatever_the_rows_hold(value):
    X = np.random.default_rng(2).normal(size=(700, 20)).astype(np.float32)
    C0 = X[:300].copy()
    X[[0, 5, 699]] = value
    _, lab, _, _ = kmeans_lloyd(X, C0, 3)
    assert lab.min() >= 0 and lab.max() < 300


@pytest.mark.gpu
def test_preservation_next_to_a_sentinel():
    rng = np.random.default_rng(3)
    X = rng.normal(size=(9000, 12)).astype(np.float32)
    Y = rng.normal(size=(9000, 3)).astype(np.float32)
    X[8999, 1], Y[0, 2] = 1e20, -1e20
    q = np.r_[0, 8999, rng.choice(8000, 60, replace=False) + 1].astype(np.int32)
    assert neighbourhood_preservation(X, Y, 15, q)[0] == mo.neighbourhood_preservation(X, Y, 15, q)[0]


@pytest.mark.gpu
@pytest.mark.parametrize("scale", [1e-20, 1e-22, 1e-24, 1e-30])
def test_neighbours_of_rows_whose_squares_underflow(scale):
    rng = np.random.default_rng(4)
    X = (scale * rng.normal(size=(400, 18))).astype(np.float32)
    c = rng.integers(0, 3, 400)
    assert np.array_equal(knn_in_clusters(X, c, 3, 5).astype(np.int64), ko.in_cluster_knn(X, c, 5)[0])
    C0 = X[:9].copy()
    C_ref, lab_ref, it_ref, _ = km.lloyd(X, C0, 3)
    C, lab, it, _ = kmeans_lloyd(X, C0, 3)
    assert it == it_ref and np.array_equal(lab.astype(np.int64), lab_ref) and np.array_equal(C, C_ref)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [5, 700])
def test_hash_planes_find_an_anchor_whatever_the_rows_hold(rows):
    rng = np.random.default_rng(5)
    X, planes = rng.normal(size=(700, 12)).astype(np.float32), rng.normal(size=(5, 12)).astype(np.float32)
    X[rng.permutation(700)[:rows], 3] = np.nan           # their projections have no place in the order
    _, buckets = kmeans_lsh_init(X, 20, planes, None, return_buckets=True)
    assert buckets.min() >= 0 and buckets.max() < 20
    Y = rng.normal(size=(9000, 3)).astype(np.float32)
    Y[::3] = np.nan                                      # slices of candidates: the merge has a place for every one of them
    q = np.arange(64, dtype=np.int32)
    assert neighbourhood_preservation(Y, Y, 5, q)[0] == 5 * 64


# ---------------------------------------------------------------- arrays that begin anywhere
@pytest.mark.gpu
@pytest.mark.parametrize("offset", [1, 2, 3])
@pytest.mark.parametrize("d", [12, 132])
def test_views_at_any_offset(d, offset):
    from paper_2505_15511_amd import random_triplet_accuracy
    rng = np.random.default_rng(d + offset)

    def shifted(a):
        t = torch.empty(a.size + 4, device="cuda")[offset:offset + a.size].view(a.shape)
        t.copy_(torch.from_numpy(a))
        assert t.data_ptr() % 16 == 4 * offset and t.is_contiguous()
        return t

    n, K = 1500, 3
    c = torch.from_numpy(rng.integers(0, 4, n).astype(np.int32)).cuda()
    Xh, Yh = rng.normal(size=(n, d)).astype(np.float32), rng.normal(size=(n, 2)).astype(np.float32)
    planes = rng.normal(size=(3, d)).astype(np.float32)
    results = []
    for put in (lambda a: torch.from_numpy(a).cuda(), shifted):
        X, Y = put(Xh), put(Yh)
        C, lab, it, inertia = kmeans_lloyd(X, put(Xh[:K].copy()), 3)
        cen, buckets = kmeans_lsh_init(X, K, put(planes), None, return_buckets=True)
        results.append([knn_in_clusters(X, c, 4, 9), C, lab, cen, buckets, pca_init(X, 0.0),
                        neighbourhood_preservation(X, Y, 7)[0], random_triplet_accuracy(X, Y, 20_000, 3)[0], it])
    for a, b in zip(*results):
        if isinstance(a, torch.Tensor) and a.shape == (n, 2):      # the scores' sums are added in another order
            assert torch.allclose(a, b, rtol=0.0, atol=1e-6 * float(a.abs().max()))
        else:
            assert torch.equal(a, b) if isinstance(a, torch.Tensor) else a == b


@pytest.mark.gpu
@pytest.mark.parametrize("size,k", [(2047, 3), (2048, 3), (2061, 16), (8195, 16), (2047, 17), (2048, 17), (2055, 32)])
def test_exact_path_by_workgroups_and_by_wavefronts(size, k):
    """A sentinel sends its whole cluster of `size` points to the exact path: too few for a wavefront each, and enough."""
    rng = np.random.default_rng(size)
    c = rng.permutation(np.repeat([0, 1], [size, 9]))
    X = rng.integers(-9, 9, size=(len(c), 5)).astype(np.float32)
    X[np.flatnonzero(c == 0)[0], 0] = 1e20
    out, stats = knn_in_clusters(X, c, 2, k, return_stats=True)
    assert size <= stats["fallback_queries"] <= size + 9
    assert np.array_equal(out.astype(np.int64), ko.in_cluster_knn(X, c, k)[0])


@pytest.mark.gpu
@pytest.mark.parametrize("n", [2047, 2048, 2100])
def test_exact_assignment_by_workgroups_and_by_wavefronts(n):
    rng = np.random.default_rng(n)
    X = rng.integers(-3, 3, size=(n, 36)).astype(np.float32)
    X[3, 0] = 1e20
    C0 = X[rng.choice(n, 300, replace=False)].copy()
    C_ref, lab_ref, it_ref, _ = km.lloyd(X, C0, 2)
    C, lab, it, _ = kmeans_lloyd(X, C0, 2)
    assert it == it_ref and np.array_equal(lab.astype(np.int64), lab_ref) and np.array_equal(C, C_ref)


# ---------------------------------------------------------------- memory kept between calls
@pytest.mark.gpu
def test_kept_memory_is_freed_on_request():
    from paper_2505_15511_amd import Nomad, release_memory, workloads
    X = torch.randn(200_000, 64, device="cuda")
    c = torch.randint(0, 50, (200_000,), device="cuda", dtype=torch.int32)
    first = knn_in_clusters(X, c, 50, 15)
    release_memory()
    free0 = torch.cuda.mem_get_info()[0]
    again = knn_in_clusters(X, c, 50, 15)
    free1 = torch.cuda.mem_get_info()[0]
    assert torch.equal(first, again) and free0 - free1 > 4 * 200_000 * 23 * 2     # candidates and keys at least are kept
    w = workloads.make_config(3, scale=0.02)
    release_memory()
    with Nomad.from_workload(w) as nm:
        held = nm.device_bytes()
        nm.set_graph(w.row_ptr, w.col_idx, w.weights, w.cluster_of, w.cluster_group)   # its own blocks, taken again
        assert held <= nm.device_bytes() <= 2 * held
        release_memory()                                                              # what the context holds stays
        nm.set_embedding(w.theta0)
        nm.epoch(0)
        theta = nm.get_embedding()
    release_memory()
    release_memory()
    assert torch.cuda.mem_get_info()[0] >= free0 and np.isfinite(theta).all()
    assert torch.equal(knn_in_clusters(X, c, 50, 15), first)
