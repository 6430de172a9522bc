"""Lloyd's iterations where some clusters gain and lose no point while others go on: only the changed ones are computed, and centroids,
labels and iterations are the oracle's, bit for bit, whenever the run is stopped."""
import numpy as np
import pytest
import torch

from oracle import kmeans_oracle as km
from paper_2505_15511_amd import kmeans_lloyd

pytestmark = pytest.mark.gpu


# sums in parallel (two widths of loads, odd rows), clusters shorter than 128 points, more than 256 centroids (two passes of the sort), as many as are marked
# in LDS and one more
@pytest.mark.parametrize("n,d,K", [(26000, 20, 24), (20001, 132, 20), (18000, 66, 30), (17001, 7, 160), (40000, 4, 300), (17100, 3, 1024), (17100, 3, 1025)])
def test_clusters_that_do_not_change_keep_their_centroids(n, d, K):
    rng = np.random.default_rng(n)
    centres = 40.0 * rng.normal(size=(K // 2, d))                       # far apart: a cluster with one centroid is settled at once
    c = rng.integers(0, K // 2, n)
    X = (centres[c] + rng.normal(size=(n, d))).astype(np.float32)
    start = centres[:K // 2 - 2]                                         # a centroid each, but for two clusters
    C0 = np.concatenate([start, start[:1] + rng.normal(size=(K - len(start) - 1, d)), 1e4 * np.ones((1, d))]).astype(np.float32)   # .. and many in one; an empty one
    for iters in (2, 3, 5, 40):
        C_ref, lab_ref, it_ref, _ = km.lloyd(X, C0, iters)
        C, lab, it, _ = kmeans_lloyd(torch.from_numpy(X).cuda(), torch.from_numpy(C0).cuda(), iters)
        assert it == it_ref and np.array_equal(lab.cpu().numpy().astype(np.int64), lab_ref)
        assert np.array_equal(C.cpu().numpy(), C_ref)
