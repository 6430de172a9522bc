"""Lloyd's iterations at the edges of their one-launch steps: sets whose sums are taken in one launch and the first that are not,
more than one chunk of columns, clusters of one stage of rows and a row more or less, centroids prepared in one launch and the
first that are not.  Everything equal to the oracle's."""
import numpy as np
import pytest

from oracle import kmeans_oracle
from paper_2505_15511_amd import kmeans_lloyd

pytestmark = pytest.mark.gpu


def run(X, C, iters):
    c, lab, it, inertia = kmeans_lloyd(X, C, iters)
    oc, olab, oit, oinertia = kmeans_oracle.lloyd(X, C, iters)
    assert it == oit and np.array_equal(lab, olab) and np.array_equal(c, oc)
    assert abs(inertia - oinertia) <= 1e-9 * abs(oinertia)


@pytest.mark.parametrize("n,d,K", [(1, 3, 1), (5, 1, 5), (2_047, 64, 3), (2_049, 65, 3), (16_384, 7, 4), (16_385, 7, 4), (900, 130, 40)])
def test_points(n, d, K):
    rng = np.random.default_rng(n + d)
    X = (rng.normal(size=(n, d)) + 3.0 * rng.integers(0, 3, size=(n, 1))).astype(np.float32)
    run(X, X[rng.permutation(n)[:K]].copy(), 6)


# the one-launch sums at their lines: the longest lists, the most workgroups, the first sets past either; more centroids than are prepared in one launch
@pytest.mark.parametrize("n,d,K", [(16_384, 5, 64), (16_385, 5, 64), (9_090, 3, 10), (9_091, 3, 10), (1_538, 3, 1), (2_100, 64, 1_024), (2_100, 65, 1_024), (4_096, 128, 512), (4_096, 129, 512),
                                   (3_000, 4, 641), (3_000, 70, 769)])
def test_lines(n, d, K):
    rng = np.random.default_rng(n + d + K)
    X = (rng.normal(size=(n, d)) + 3.0 * rng.integers(0, 3, size=(n, 1))).astype(np.float32)
    run(X, X[rng.permutation(n)[:K]].copy(), 3)


@pytest.mark.parametrize("m", [63, 64, 65, 128])
def test_stages_of_rows(m):
    """Two clusters of m rows far apart, and a third centroid that stays empty."""
    rng = np.random.default_rng(m)
    X = rng.normal(size=(2 * m, 10)).astype(np.float32)
    X[::2] += 100.0
    run(X, np.stack([X[0], X[1], np.full(10, -1e4, np.float32)]), 5)


@pytest.mark.parametrize("K", [128, 129])
def test_centroids(K):
    """128 x 512 values are prepared in one launch, one row more are not."""
    rng = np.random.default_rng(K)
    X = rng.normal(size=(600, 512)).astype(np.float32)
    run(X, X[:K].copy(), 3)


def test_stops_when_nothing_moves():
    """The host runs an iteration ahead; count, labels and centroids are those of the iteration that moved nothing."""
    rng = np.random.default_rng(0)
    X = (rng.normal(size=(3_000, 5)) + 50.0 * rng.integers(0, 4, size=(3_000, 1))).astype(np.float32)
    for iters in (1, 2, 3, 4, 50):
        run(X, X[:4].copy(), iters)
