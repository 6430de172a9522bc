"""The neighbour filter far into a long group: the small products only where a lane may still pass.  GPU."""
import numpy as np
import pytest
import torch

from oracle import knn_oracle as ko
from paper_2505_15511_amd import knn_in_clusters

pytestmark = pytest.mark.gpu


# (n, d, k): 32-row tiles with short lists (sifting from row 512 (k + 8) on) just at the line, one row past it and far beyond it,
# with two and with eight wavefronts a workgroup; long lists; 16-row tiles (from row 128 (k + 8) on) with both list lengths
@pytest.mark.parametrize("n,d,k", [(11776, 20, 15), (11777, 20, 15), (9000, 128, 5), (34001, 40, 15), (33333, 128, 1), (33000, 10, 12), (34000, 64, 20),
                                   (18001, 300, 15), (17000, 200, 20), (5003, 768, 15)])
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
