"""Points whose nearest centroid the filter leaves open, in bulk (ties, near duplicates), where a wavefront takes two tiles of them, three or the most,
in rows that are in the order of their classes: labels and centroids are the oracle's, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import kmeans_oracle as km
from paper_2505_15511_amd import kmeans_lloyd

pytestmark = pytest.mark.gpu


# 32- and 16-row tiles; the last tile short of rows, and short of tiles for the last wavefronts
@pytest.mark.parametrize("n,d,K", [(16385, 7, 40), (20001, 20, 9), (65569, 3, 5), (131073, 2, 4), (983041, 2, 3), (17000, 260, 12), (32785, 300, 4), (33000, 513, 3)])
def test_points_that_are_left_open(n, d, K):
    rng = np.random.default_rng(n)
    X = rng.integers(0, 2, (n, d)).astype(np.float32)
    X[:n // 3] = X[0]                                        # one class first: all of its points are open, or none
    C0 = X[rng.choice(n, K, replace=False)].copy()
    C0[K // 2] = C0[0]                                       # a centroid twice: the first of the two has the points
    C0[K - 1, 0] = np.nextafter(C0[K - 1, 0], np.float32(2))
    lab_ref, dist_ref = km.assign(X, C0)
    C, lab, it, inertia = kmeans_lloyd(torch.from_numpy(X).cuda(), torch.from_numpy(C0.copy()).cuda(), 1)
    assert it == 1 and np.array_equal(lab.cpu().numpy().astype(np.int64), lab_ref)
    assert np.array_equal(C.cpu().numpy(), km.update(X, lab_ref, C0))
    assert abs(inertia - dist_ref.sum()) <= 1e-12 * dist_ref.sum()
