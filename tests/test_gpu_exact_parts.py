"""Few flagged queries: their groups are cut into parts that several workgroups walk.  GPU."""
import numpy as np
import pytest
import torch

from oracle import knn_oracle as ko
from paper_2505_15511_amd import knn_in_clusters

pytestmark = pytest.mark.gpu


# `copies` copies of one row: more ties than the filter's list holds, so each of them is flagged (one query's group cut into the
# most parts; a few; each into two or three; more than half as many as workgroups, where nothing is cut any longer)
@pytest.mark.parametrize("copies", [26, 60, 150, 257])
@pytest.mark.parametrize("sizes,d,k", [([9000, 700], 40, 15), ([2500, 1100], 20, 1), ([5000], 7, 32), ([1030, 1023, 1025], 300, 16), ([600, 600], 64, 17)])
def test_flagged_queries_are_exact(copies, sizes, d, k):
    print(f"copies={copies} sizes={sizes} d={d} k={k}", flush=True)
    rng = np.random.default_rng(copies + d)
    c = np.repeat(np.arange(len(sizes)), sizes)
    X = rng.normal(size=(len(c), d)).astype(np.float32)
    where = np.sort(rng.choice(sizes[0], copies, replace=False))
    X[where] = X[where[0]]
    far_tie = len(sizes) > 1 and copies < 150            # an exact tie far away, in another group
    if far_tie:
        where2 = sizes[0] + np.arange(k + 12)
        X[where2] = X[where2[0]]
    perm = rng.permutation(len(c))
    X, c = X[perm], c[perm]
    out, st = knn_in_clusters(torch.from_numpy(X).cuda(), torch.from_numpy(c.astype(np.int32)).cuda(), len(sizes), k, return_stats=True)
    print(f"  flagged {st['fallback_queries']}", flush=True)
    ties = (copies if copies > k + 8 else 0) + (k + 12 if far_tie else 0)   # (a list holds k + 8: fewer copies than that may be told apart)
    # up to 256 queries, half as many as workgroups, are cut (points near the copies are flagged too: their k-th neighbour is a tie)
    assert ties <= st["fallback_queries"] <= (256 if copies < 256 else 512)
    ref, _ = ko.in_cluster_knn(X, c, k)
    assert np.array_equal(out.cpu().numpy().astype(np.int64), ref)


def test_group_of_more_rows_than_the_most_parts_have_lanes():
    """Rows for 33 times four a lane and few flagged queries: the most parts, each walked in more than one pass."""
    n, d, k, copies = 33 * 1024 * 4 + 5, 8, 1, 11
    rng = np.random.default_rng(3)
    X = rng.normal(size=(n, d)).astype(np.float32)
    where = np.sort(rng.choice(n, copies, replace=False))
    X[where] = X[where[0]]
    out, st = knn_in_clusters(torch.from_numpy(X).cuda(), torch.zeros(n, dtype=torch.int32, device="cuda"), 1, k, return_stats=True)
    assert copies <= st["fallback_queries"] <= 16                           # (of 512 workgroups)
    some = np.concatenate([where, rng.choice(n, 40, replace=False)])
    D = ko.pair_distances(X[some], X)
    D[np.arange(len(some)), some] = np.inf
    assert np.array_equal(out.cpu().numpy()[some].astype(np.int64), np.argsort(D, axis=1, kind="stable")[:, :k])
