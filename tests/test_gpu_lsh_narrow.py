"""Hash start: one, two or four wavefronts share 64 rows, by rows, columns and planes; about the edges of workgroups and columns in each, against the oracle bit for bit."""
import numpy as np
import pytest

from oracle import kmeans_oracle as km
from paper_2505_15511_amd import kmeans_lsh_init

pytestmark = pytest.mark.gpu


def check(n, K, d, n_planes=None):
    rng = np.random.default_rng(n + 10 * d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    X[n // 2:] = np.round(X[n // 2:])                   # rows on planes through rows
    planes = rng.standard_normal((n_planes or max(1, int(np.ceil(np.log2(K)))), d)).astype(np.float32)
    planes[0] = np.sign(planes[0])
    anchors = rng.integers(0, n, len(planes)).astype(np.int32)
    C_ref, buckets_ref = km.lsh_init(X, planes, anchors, K)
    C, buckets = kmeans_lsh_init(X, K, planes, anchors, return_buckets=True)
    assert np.array_equal(buckets, buckets_ref) and np.array_equal(C, C_ref)


@pytest.mark.parametrize("d", [1, 2, 15, 16, 17, 31, 32, 33, 49])
@pytest.mark.parametrize("n,K", [(255, 2), (256, 200), (257, 250), (129, 100), (700, 300)])
def test_few_rows(n, K, d):
    check(n, K, d)


@pytest.mark.parametrize("n,d,n_planes", [(140_001, 31, 12), (140_001, 33, 12), (140_001, 32, 8), (270_017, 31, 8), (270_017, 33, 5), (66_000, 65, 9), (66_000, 63, 9), (70_003, 31, 20), (70_003, 32, 30)])
def test_many_rows(n, d, n_planes):
    check(n, 24, d, n_planes)
