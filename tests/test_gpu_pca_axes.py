"""The axes of few columns: widths at the edges of the compiled sizes (a multiple of 32 columns and one more or less, whole and ragged
16-row tiles), full rank and columns that vanish or repeat others; scores against the oracle's.  The bound is the other PCA tests':
an axis errs by the residual (1e-12) over the spectral gap."""
import numpy as np
import pytest

from oracle import pca_oracle
from paper_2505_15511_amd import pca_init

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [3, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 112, 113, 127, 128])
@pytest.mark.parametrize("kind", ["full", "zeros", "copies", "tiny"])
def test_widths(d, kind):
    rng = np.random.default_rng(d)
    X = rng.normal(size=(600, d)) * np.linspace(1.0, 0.2, d)
    X[:, 0] *= 4.0                      # gaps above the second and the third axis
    X[:, 1] *= 2.0
    if kind == "zeros":
        X[:, 2:] = 0.0
    elif kind == "copies":
        X[:, 2:] = X[:, np.arange(d - 2) % 2] * 0.25
    elif kind == "tiny":
        X *= 1e-30
    X = X.astype(np.float32)
    theta, ref = pca_init(X, 0.01), pca_oracle.pca_init(X, 0.01)
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert np.abs(np.asarray(theta, np.float64) - ref).max() <= 1e-5 * np.abs(ref).max()
