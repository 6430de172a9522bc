"""The inertia of nomad_kmeans_lloyd: every row counted once, at the edges of its workgroups' rows and rounds, in rows of every alignment.
Reference: float64 sums; n additions in any order are off by n 2^-53 of the sum at most, here below 1e-10."""
import numpy as np
import pytest
import torch

from paper_2505_15511_amd import kmeans_lloyd

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 64, 65, 255, 256, 257, 512 * 256 - 1, 512 * 256, 512 * 256 + 1, 512 * 256 + 300])
@pytest.mark.parametrize("d", [1, 4, 67, 68])
def test_every_row_counts_once(n, d):
    g = torch.Generator().manual_seed(n + d)
    X = torch.randn(n, d, generator=g)
    X[-1] *= 100.0                                           # the last row decides the sum: it is there, and no other row in its place
    C0 = X[:1].clone()
    _, _, it, inertia = kmeans_lloyd(X.cuda(), C0.clone().cuda(), 1)
    ref = float(((X.double() - C0.double()) ** 2).sum())
    assert it == 1 and abs(inertia - ref) <= 1e-10 * ref
