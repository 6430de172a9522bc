"""The covariance about a shift taken from a sample of the rows: sets smaller and larger than the sample, every number of column
tiles up to three, rows in cluster order far from the origin, and an outlier among the sampled rows; scores against the oracle's."""
import numpy as np
import pytest

from oracle import pca_oracle
from paper_2505_15511_amd import pca_init

pytestmark = pytest.mark.gpu


def data(n, d, seed, offset=0.0, outlier=0.0):
    rng = np.random.default_rng(seed)
    X = rng.normal(size=(n, d)) * np.linspace(1.0, 0.1, d)
    X[:, 0] *= 3.0                                                   # a gap above the third axis
    X[:, 1] *= 2.0
    X += offset + 5.0 * (np.arange(n) * 4 // n)[:, None] * rng.normal(size=d)   # four clusters, in order
    X[0] += outlier                                                  # row 0 is always sampled
    return X.astype(np.float32)


@pytest.mark.parametrize("n,d", [(2, 2), (255, 16), (256, 17), (257, 64), (1_000, 65), (5_000, 128), (3_000, 129), (700, 190)])
@pytest.mark.parametrize("offset,outlier", [(0.0, 0.0), (1_000.0, 0.0), (-50.0, 300.0)])
def test_scores(n, d, offset, outlier):
    X = data(n, d, n + d, offset, outlier)
    theta = pca_init(X, 0.01)
    theta = theta[0] if isinstance(theta, tuple) else theta
    ref = pca_oracle.pca_init(X, 0.01)
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert np.abs(np.asarray(theta, np.float64) - ref).max() <= 1e-5 * np.abs(ref).max()
