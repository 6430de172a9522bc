"""Which of the two edge passes of sorted forces runs (nomad_edges_in_runs): the comparison of forces in runs with records in chains is one of two different passes, and a
pass that could not be set up is named."""
import pytest
import torch

import tests.test_gpu_runs as runs
from paper_2505_15511_amd import EDGES_EXCHANGED, EDGES_LDS_SUMS, EDGES_RECORDS, SCATTER_ATOMIC, Nomad, release_memory
from tests.test_gpu_exchange import graph

pytestmark = pytest.mark.gpu
# points, negatives, edges (several blocks, the last one ragged), lanes of a segment of the sums
LANES = [(60_000, 0, 7 * 1536 + 77, 8), (900_001, 0, 500_000, 8), (3_000_000, 2, 40_003, 8), (900_001, 1, 500_001, 16), (900_001, 8, 70_001, 16), (40_000, 8, 70_000, 16),
         (100_000, 5, 300_001, 32), (900_001, 4, 500_000, 32), (200_000, 2, 100_003, 16), (900_001, 5, 200_001, 32), (4_100, 5, 9_000, 32)]


@pytest.fixture(autouse=True)
def told(monkeypatch):
    """Every context of the comparison says which pass it runs, and both sides occur."""
    seen = set()

    class Told(Nomad):
        def __init__(self, *args, tune=None, **kw):
            super().__init__(*args, tune=tune, **kw)
            self.chains = "record_sort" in tune

        def set_graph(self, *args):
            assert not self.edges_in_runs()
            super().set_graph(*args)
            assert self.edges_in_runs() == (not self.chains)
            seen.add(self.chains)

    monkeypatch.setattr(runs, "Nomad", Told)
    return seen


@pytest.mark.parametrize("kind", ["plain", "groups", "far"])
@pytest.mark.parametrize("s", range(9))
def test_blocks(s, kind, told):
    runs.both(2_000, s, *graph(2_000, runs.BLOCK[s] + 77, s), kind=kind)
    assert told == {False, True}


@pytest.mark.parametrize("n,s,E,lanes", LANES)
def test_lanes(n, s, E, lanes, told):
    runs.both(n, s, *graph(n, E, s))
    assert told == {False, True}


@pytest.mark.parametrize("n,E,s,kind", [(12_000, 3_000, 2, "plain"), (20_000, 32_768, 1, "groups"), (200_000, 5_000, 5, "plain"), (900_001, 20_000, 0, "far")])
def test_sparse_graphs_are_left_to_chains(n, E, s, kind):
    cluster_of = (torch.arange(n, device="cuda") * 7 // n).to(torch.int32)
    row_ptr, col, theta = graph(n, E, s)
    got = []
    for tune in ({}, {"exchange": 2}, {"record_sort": 1}):
        with Nomad(n, 7, s, 5.0, 10, 1.0, 7, sampled_far_field=kind == "far", tune=tune) as nm:
            nm.set_graph(row_ptr, col, None, cluster_of, None if kind == "plain" else torch.arange(7, dtype=torch.int32, device="cuda"))
            assert not nm.edges_in_runs() and nm.edge_pass() == EDGES_RECORDS and nm.note() == ""
            nm.set_embedding(theta)
            nm.epoch(0)
            got.append((nm.get_gradient(device=True), nm.get_embedding(device=True)))
    runs.same(got[0], got[2]), runs.same(got[1], got[2])


@pytest.mark.parametrize("n,want,kw", [(2_000, EDGES_LDS_SUMS, {}), (20_000, EDGES_RECORDS, {}), (1_000_000, EDGES_EXCHANGED, {}), (20_000, None, {"scatter_mode": SCATTER_ATOMIC})])
def test_other_passes_are_not_in_runs(n, want, kw):
    row_ptr, col, _ = graph(n, 50_000, 3)
    with Nomad(n, 1, 5, 5.0, 10, 1.0, 7, **kw) as nm:
        nm.set_graph(row_ptr, col, None, torch.zeros(n, dtype=torch.int32, device="cuda"))
        assert nm.edges_in_runs() == (want == EDGES_RECORDS) and (want is None or nm.edge_pass() == want) and nm.note() == ""


def test_a_pass_that_could_not_be_set_up_is_named():
    """Forces in runs count their slots in 32 bits: 712 M edges in one phase have more.  (Only set up: nothing of this runs.)"""
    n, degree = 300_000, 2_375
    col = torch.arange(n, dtype=torch.int32, device="cuda")[:, None] + torch.arange(1, degree + 1, dtype=torch.int32, device="cuda")[None]
    col = col.remainder_(n).reshape(-1)
    row_ptr = torch.arange(n + 1, dtype=torch.int32, device="cuda") * degree
    with Nomad(n, 1, 5, 5.0, 10, 1.0, 7, tune={"record_phases": 1}) as nm:
        nm.set_graph(row_ptr, col, None, torch.zeros(n, dtype=torch.int32, device="cuda"))
        assert not nm.edges_in_runs() and nm.edge_pass() == EDGES_RECORDS
        assert "forces in runs could not be set up (size out of range)" in nm.note()
    del col, row_ptr
    release_memory()
    torch.cuda.empty_cache()
