"""knn_in_clusters where the rows of a cluster are laid out cell by cell (long clusters of wide rows): the order has no part in
the answer.  Reference: the oracle's float64 distances, bit for bit, on sampled queries."""
import numpy as np
import pytest
import torch

from oracle import knn_oracle as ko
from paper_2505_15511_amd import knn_in_clusters

pytestmark = pytest.mark.gpu


def _rows(kind, n, d, clusters, seed):
    rng = np.random.default_rng(seed)
    c = rng.integers(0, clusters, n).astype(np.int32)
    if kind == "grid":                                   # ties in bulk
        return rng.integers(0, 2, (n, d)).astype(np.float32), c
    X = rng.normal(size=(n, d)).astype(np.float32)
    if kind == "components":                             # four components a cluster, as far apart as their points are
        X += rng.normal(size=(4 * clusters, d)).astype(np.float32)[4 * c + rng.integers(0, 4, n)]
    elif kind == "duplicates":                           # fewer different rows than cells
        X = X[rng.integers(0, 7, n)]
    return X, c


# every tile shape, list class and number of wavefronts; mean cluster on both sides of 200,000 / d
@pytest.mark.parametrize("kind,n,d,clusters,k", [
    ("components", 3100, 70, 1, 15), ("components", 2000, 128, 1, 8), ("components", 4100, 201, 3, 20), ("components", 2100, 256, 2, 15),
    ("components", 900, 300, 1, 10), ("components", 1100, 600, 2, 15), ("components", 1300, 768, 3, 32), ("components", 1600, 130, 1, 30),
    ("noise", 1700, 127, 1, 32), ("grid", 1200, 200, 1, 15), ("duplicates", 1500, 160, 1, 15), ("components", 780, 512, 2, 5),
    ("components", 772, 517, 2, 24),                     # one row short of the order
    ("components", 34000, 16, 2, 15), ("components", 34000, 61, 7, 9), ("components", 34000, 96, 16, 15), ("noise", 34000, 126, 20, 31),
    ("components", 17000, 300, 25, 15), ("components", 17000, 190, 16, 25), ("components", 33000, 12, 1, 32),
    # twelve and sixteen wavefronts a workgroup, which take a little more than one round of eight to be worth it (tests/test_filter_plan.py), ordered and not
    ("components", 70000, 16, 17, 15), ("noise", 70000, 30, 17, 8), ("grid", 70000, 15, 17, 15), ("components", 70000, 61, 17, 9), ("components", 70000, 40, 17, 15),
    ("components", 70000, 90, 17, 15), ("components", 70000, 128, 17, 10), ("components", 70000, 12, 17, 32), ("noise", 70000, 31, 17, 20), ("components", 36000, 300, 9, 15),
    ("components", 36000, 260, 9, 5), ("components", 36000, 130, 9, 25), ("components", 36000, 200, 9, 20), ("components", 70000, 64, 17, 30), ("components", 65536, 64, 17, 30)])
def test_the_order_of_the_rows_has_no_part_in_the_answer(kind, n, d, clusters, k):
    X, c = _rows(kind, n, d, clusters, n + d)
    out = knn_in_clusters(torch.from_numpy(X).cuda(), torch.from_numpy(c).cuda(), clusters, k).cpu().numpy()
    rng = np.random.default_rng(1)
    for r in range(min(clusters, 3)):
        members = np.nonzero(c == r)[0]
        q = np.concatenate([rng.choice(len(members), min(len(members), 150), replace=False), [0, len(members) - 1]])
        D = ko.pair_distances(X[members[q]], X[members])
        D[np.arange(len(q)), q] = np.inf
        ref = members[np.argsort(D, axis=1, kind="stable")[:, :k]]
        assert np.array_equal(out[members[q]], ref), (kind, r)
    # the whole answer: other points of the same cluster, none twice
    assert (c[out] == c[:, None]).all() and (out != np.arange(n)[:, None]).all()
    s = np.sort(out, axis=1)
    assert (s[:, 1:] != s[:, :-1]).all()


def test_rows_that_are_not_aligned_and_clusters_of_any_size():
    rng = np.random.default_rng(3)
    sizes = [1, 2, 15, 16, 17, 0, 40, 3000]
    c = np.repeat(np.arange(len(sizes)), sizes).astype(np.int32)
    c = c[rng.permutation(len(c))]
    n, d, k = len(c), 640, 15
    X = rng.normal(size=(n, d)).astype(np.float32)
    ref, _ = ko.in_cluster_knn(X, c, k, block=64)
    store = torch.zeros(n * d + 1, device="cuda")
    view = store[1:].view(n, d)                          # rows that begin 4 bytes past a boundary of 16
    view.copy_(torch.from_numpy(X))
    for rows in (torch.from_numpy(X).cuda(), view):
        out = knn_in_clusters(rows, torch.from_numpy(c).cuda(), len(sizes), k)
        assert np.array_equal(out.cpu().numpy().astype(np.int64), ref)
