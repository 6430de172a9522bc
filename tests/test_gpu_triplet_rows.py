"""Triplets whose rows the wavefront reads together (32 columns and more): ragged ends, unaligned rows.  GPU."""
import numpy as np
import pytest
import torch

from oracle import metrics_oracle as mo
from paper_2505_15511_amd import random_triplet_accuracy

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [31, 32, 33, 36, 63, 64, 65, 97, 128, 130, 257])
@pytest.mark.parametrize("shift", [0, 1])      # float32 values by which the rows begin off a 16-byte boundary
def test_counts_are_exact(d, shift):
    print(f"triplets d={d} shift={shift}", flush=True)
    n, T = 513, 64 * 37 + 1
    rng = np.random.default_rng(d)
    X = rng.integers(-2, 3, size=(n, d)).astype(np.float32) + (rng.random((n, d)) < 0.1).astype(np.float32) * 1e-3     # ties and near ties
    Y = X[:, :2].copy()
    buf = torch.zeros(n * d + shift, device="cuda")
    Xd = buf[shift:].view(n, d)
    Xd.copy_(torch.from_numpy(X))
    ref = mo.random_triplet_accuracy(X, Y, T, seed=5)[0]
    assert random_triplet_accuracy(Xd, torch.from_numpy(Y).cuda(), T, 5)[0] == ref
