"""The loss with a position a lane against the loss with sixteen lanes a row, which problems with atomic scatter take: the terms are the same, and none is
negative, so two orders of summing E of them in float64 agree to 2 E 2^-53 of their sum."""
import pytest
import torch

from paper_2505_15511_amd import SCATTER_ATOMIC, SCATTER_DETERMINISTIC, Nomad
from tests.test_gpu_exchange import graph

pytestmark = pytest.mark.gpu


def loss(n, s, row_ptr, col, theta, kind, weights, mode):
    clusters = 1 if kind == "plain" else min(n, 7)
    cluster_of = (torch.arange(n, device="cuda") * clusters // n).to(torch.int32)
    groups = None if kind == "plain" else torch.arange(clusters, dtype=torch.int32, device="cuda")
    nm = Nomad(n, clusters, s, 5.0, 10, 1.0, 77, scatter_mode=mode, sampled_far_field=kind == "far")
    nm.set_graph(row_ptr, col, weights, cluster_of, groups)
    nm.set_embedding(theta)
    return nm.loss(3)


@pytest.mark.parametrize("kind", ["plain", "groups", "far"])
@pytest.mark.parametrize("s", [0, 1, 4, 5, 8, 9])
@pytest.mark.parametrize("n,E", [(2, 1), (17, 255), (17, 256), (2_000, 257), (2_000, 2_049), (20, 100_000), (30_001, 600_011), (524_288, 700_001), (524_289, 700_001)])
def test_loss(n, E, s, kind):
    row_ptr, col, theta = graph(n, E, E + s)
    weights = torch.rand(E, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda") + 0.1 if s == 4 else None
    got, want = (loss(n, s, row_ptr, col, theta, kind, weights, mode) for mode in (SCATTER_DETERMINISTIC, SCATTER_ATOMIC))
    assert want > 0 or (s == 0 and want >= 0)
    assert abs(got - want) <= 2.0 * E * 2.0**-53 * abs(want)
