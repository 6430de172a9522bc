"""The edge pass that sums in LDS against the one that sorts records: the same bits, for one population, groups and the sampled far field."""
import pytest
import torch

from paper_2505_15511_amd import EDGES_LDS_SUMS, EDGES_RECORDS, Nomad
from tests.test_gpu_exchange import graph, same

pytestmark = pytest.mark.gpu


def epochs(n, s, args, tune, R=1, groups=None, n_epochs=2, **kw):
    row_ptr, col, theta = args
    nm = Nomad(n, R, s, 5.0, 10, 1.0, 77, tune=tune, **kw)
    cluster = (torch.arange(n, device="cuda") * R // n).to(torch.int32)
    nm.set_graph(row_ptr, col, None, cluster, groups)
    assert nm.edge_pass() == (EDGES_RECORDS if tune else EDGES_LDS_SUMS) and nm.note() == ""
    nm.set_embedding(theta)
    for t in range(n_epochs):
        nm.epoch(t)
    return nm.get_gradient(device=True), nm.get_embedding(device=True)


def both(n, s, args, **kw):
    same(epochs(n, s, args, None, **kw), epochs(n, s, args, {"record_sort": 1}, **kw))


@pytest.mark.parametrize("s", range(0, 9))
@pytest.mark.parametrize("E", [1, 1_023, 1_024, 1_025, 40_000])
def test_rounds(s, E):
    both(1_500, s, graph(1_500, E, 10 * s + E % 7, hub=E // 4))


@pytest.mark.parametrize("n", [2, 31, 32, 33, 1_000, 10_224])
def test_points(n):
    both(n, 5, graph(n, 300_000, n))


@pytest.mark.parametrize("s", [1, 2, 5, 8])
@pytest.mark.parametrize("kw", [{}, {"sampled_far_field": True}, {"batches_per_epoch": 3}], ids=["means", "sampled means", "sub-steps"])
def test_groups(s, kw):
    groups = torch.tensor([0, 0, 1, 2, 2, 2, 3], dtype=torch.int32, device="cuda")
    both(3_333, s, graph(3_333, 50_000, s), R=7, groups=groups, **kw)


def test_more_edges_than_workgroups_take_in_one_round():
    both(9_000, 5, graph(9_000, 2_000_000, 3, hub=50_000))
