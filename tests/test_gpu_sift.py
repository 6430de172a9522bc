"""The neighbour filter far into a long group: the small products only where a lane may still pass.  GPU."""
import numpy as np
import pytest
import torch

from oracle import knn_oracle as ko
from paper_2505_15511_amd import knn_in_clusters

pytestmark = pytest.mark.gpu


# (n, d, k): 32-row tiles with short lists, eight wavefronts a workgroup (from 32,768 rows on; sifting from row 512 (k + 8) on) and two (from row
# 2,048 (k + 8) on: just at the line, one row past it, beyond it); long lists; 16-row tiles with both list lengths, eight wavefronts (from
# 16,384 rows on; sifting from row 128 (k + 8) on) and four (from row 512 (k + 8) on: at the line, past it)
@pytest.mark.parametrize("n,d,k", [(11776, 20, 15), (11777, 20, 15), (9000, 128, 5), (34001, 40, 15), (33333, 128, 1), (33000, 10, 12), (34000, 64, 20),
                                   (18001, 300, 15), (17000, 200, 20), (5003, 768, 15),
                                   (26624, 20, 5), (26625, 20, 5), (30001, 128, 5), (11776, 300, 15), (11777, 300, 15), (15001, 400, 15), (16301, 200, 20)])
@pytest.mark.parametrize("outlier", [False, True])
def test_neighbours_late_in_a_long_group(n, d, k, outlier):
    print(f"n={n} d={d} k={k} outlier={outlier}", flush=True)
    rng = np.random.default_rng(n + d)
    X = (3.0 * rng.normal(size=(40, d))[rng.integers(0, 40, n)] + rng.normal(size=(n, d))).astype(np.float32)
    # the nearest neighbours of the first rows are the last rows, a hair away, in bulk
    m = 3 * k
    X[n - m:] = X[rng.integers(0, 4, m)] + (1e-3 * rng.normal(size=(m, d))).astype(np.float32)
    if outlier:
        X[n // 2] *= 300.0          # scales the whole group: the small products' bound is far wider than most keys' distance
    out = knn_in_clusters(torch.from_numpy(X).cuda(), torch.zeros(n, dtype=torch.int32, device="cuda"), 1, k).cpu().numpy()
    q = np.unique(np.concatenate([np.arange(4), np.arange(n - m, n), rng.integers(0, n, 40), [n // 2]]))
    D = ko.pair_distances(X[q], X)
    D[np.arange(len(q)), q] = np.inf
    assert np.array_equal(out[q].astype(np.int64), np.argsort(D, axis=1, kind="stable")[:, :k])


@pytest.mark.parametrize("d,k", [(16, 15), (40, 20), (140, 30), (300, 10)])
def test_a_key_of_zero_keeps_its_position(d, k):
    """A row that is its group's mean has the key 0 for every query: the smallest numbers a list's entries can be."""
    print(f"d={d} k={k}", flush=True)
    rng = np.random.default_rng(d)
    half = rng.integers(-60, 61, size=(700, d)).astype(np.float32)
    half[:20] = np.sign(half[:20]) * (np.abs(half[:20]) > 45)        # a few rows close to the middle: it is among their nearest
    X = np.concatenate([half, -half, np.zeros((1, d), np.float32)])
    X = X[rng.permutation(len(X))]
    out, st = knn_in_clusters(torch.from_numpy(X).cuda(), torch.zeros(len(X), dtype=torch.int32, device="cuda"), 1, k, return_stats=True)
    print(f"  flagged {st['fallback_queries']}", flush=True)
    ref, _ = ko.in_cluster_knn(X, np.zeros(len(X), np.int32), k)
    assert np.array_equal(out.cpu().numpy().astype(np.int64), ref)
