"""Lloyd's iterations whose filter multiplies the high halves alone where these decide for nearly all points: labels, centroids and iterations are the
oracle's, bit for bit, where they decide, where they leave most points open, and where that changes from step to step."""
import numpy as np
import pytest
import torch

from oracle import kmeans_oracle as km
from paper_2505_15511_amd import kmeans_lloyd

pytestmark = pytest.mark.gpu


def _case(kind, n, d, K, rng):
    centres = (30.0 if kind == "tight" else 4.0) * rng.normal(size=(K // 4, d))
    X = centres[rng.integers(0, K // 4, n)] + (1e-2 if kind == "tight" else 1.0) * rng.normal(size=(n, d))   # tight: all of a cluster's points and centroids alike to float16
    if kind == "tails":
        X *= np.exp(rng.normal(size=(n, 1)))
    if kind == "grid":
        X = rng.integers(0, 3, (n, d))
    X = X.astype(np.float32)
    C0 = X[rng.choice(n, K, replace=False)].copy()
    if kind == "spread":                                    # far off at first: the centroids come in by and by
        C0 = (8.0 * C0).astype(np.float32)
    return X, C0


# 32- and 16-row tiles, every number of steps once; centroids in one tile and in several, not a multiple of a stage; one point below the line
@pytest.mark.parametrize("kind,n,d,K", [
    ("plain", 66000, 16, 40), ("plain", 65537, 31, 33), ("plain", 66000, 64, 36), ("plain", 65540, 90, 20), ("plain", 66001, 128, 21), ("spread", 66000, 190, 9),
    ("plain", 65536, 250, 8), ("plain", 65600, 300, 8), ("spread", 65600, 500, 5), ("plain", 65600, 765, 4), ("tight", 66000, 40, 32), ("tight", 65536, 300, 8),
    ("tails", 66000, 24, 64), ("grid", 66000, 5, 30), ("plain", 65535, 20, 16), ("spread", 70000, 9, 50)])
def test_what_the_large_products_decide(kind, n, d, K):
    X, C0 = _case(kind, n, d, K, np.random.default_rng(n + d))
    for iters in (2, 4):
        C_ref, lab_ref, it_ref, _ = km.lloyd(X, C0, iters)
        C, lab, it, _ = kmeans_lloyd(torch.from_numpy(X).cuda(), torch.from_numpy(C0).cuda(), iters)
        assert it == it_ref and np.array_equal(lab.cpu().numpy().astype(np.int64), lab_ref)
        assert np.array_equal(C.cpu().numpy(), C_ref)
