"""The edge pass that leaves its forces in runs against the one that leaves records in chains: the same lanes take the same edges, products are
rounded alike and forces are summed as integers, so gradient and embedding agree bit for bit."""
import pytest
import torch

from paper_2505_15511_amd import EDGES_RECORDS, Nomad
from tests.test_gpu_exchange import graph, same

pytestmark = pytest.mark.gpu
BLOCK = {s: 1536 if s <= 2 else 1024 if s <= 6 else 512 for s in range(9)}     # positions of a block


def epochs(n, s, row_ptr, col, theta, chains, kind="plain", tune=None, weights=None, **kw):
    clusters = 1 if kind == "plain" else min(n, 7)
    cluster_of = (torch.arange(n, device="cuda") * clusters // n).to(torch.int32)
    groups = None if kind == "plain" else torch.arange(clusters, dtype=torch.int32, device="cuda")
    nm = Nomad(n, clusters, s, 5.0, 10, 1.0, 77, tune=dict(tune or {}, **({"record_sort": 1} if chains else {"exchange": 2})), sampled_far_field=kind == "far", **kw)
    nm.set_graph(row_ptr, col, weights, cluster_of, groups)
    assert nm.edge_pass() == EDGES_RECORDS and nm.note() == ""
    nm.set_embedding(theta)
    for t in range(2):
        nm.epoch(t)
    return nm.get_gradient(device=True), nm.get_embedding(device=True)


def both(*args, **kw):
    same(epochs(*args, chains=False, **kw), epochs(*args, chains=True, **kw))


@pytest.mark.parametrize("kind", ["plain", "groups", "far"])
@pytest.mark.parametrize("s", range(9))
def test_blocks(s, kind):
    for blocks, edges in [(0, 1), (1, -1), (1, 0), (1, 1), (9, 77)]:
        E = blocks * BLOCK[s] + edges
        both(2_000, s, *graph(2_000, E, 100 * s + E % 97, hub=5_000 if blocks == 9 else 0), kind=kind)


@pytest.mark.parametrize("kind", ["plain", "groups", "far"])
@pytest.mark.parametrize("n", [2, 17, 4_097, 65_536, 300_001])
def test_points(n, kind):
    both(n, 5, *graph(n, 40_000, n), kind=kind)


# 8, 16 and 32 lanes a segment of the sums
@pytest.mark.parametrize("n,s,E", [(900_001, 1, 500_000), (900_001, 4, 500_000), (900_001, 8, 500_000), (40_000, 8, 70_000)])
def test_lanes(n, s, E):
    both(n, s, *graph(n, E, s))


@pytest.mark.parametrize("kind", ["plain", "groups", "far"])
def test_phases_sub_steps_and_weights(kind):
    n, E = 30_000, 200_003
    row_ptr, col, theta = graph(n, E, 5)
    weights = torch.rand(E, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda") + 0.1
    both(n, 5, row_ptr, col, theta, kind=kind, weights=weights)
    same(epochs(n, 5, row_ptr, col, theta, chains=False, kind=kind, tune={"record_phases": 3}), epochs(n, 5, row_ptr, col, theta, chains=True, kind=kind))
    both(n, 2, row_ptr, col, theta, kind=kind, batches_per_epoch=7)
