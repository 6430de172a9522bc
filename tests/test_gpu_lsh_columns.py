"""Hash start: a workgroup's wavefronts take sixteen of every 64 columns; rows, columns and planes about their edges, against the oracle bit for bit."""
import numpy as np
import pytest

from oracle import kmeans_oracle as km
from paper_2505_15511_amd import kmeans_lsh_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,K", [(63, 1, 2), (64, 15, 3), (65, 16, 4), (130, 17, 9), (257, 63, 20), (300, 64, 33), (511, 65, 100), (200, 129, 150), (190, 768, 17)])
def test_buckets(n, d, K):
    rng = np.random.default_rng(n + d)
    X = rng.standard_normal((n, d)).astype(np.float32)
    X[n // 2:] = np.round(X[n // 2:])                   # rows on planes through rows
    planes = rng.standard_normal((max(1, int(np.ceil(np.log2(K)))), d)).astype(np.float32)
    planes[0] = np.sign(planes[0])
    anchors = rng.integers(0, n, len(planes)).astype(np.int32)
    C_ref, buckets_ref = km.lsh_init(X, planes, anchors, K)
    C, buckets = kmeans_lsh_init(X, K, planes, anchors, return_buckets=True)
    assert np.array_equal(buckets, buckets_ref) and np.array_equal(C, C_ref)
