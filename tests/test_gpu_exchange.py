"""The exchanged edge pass against the sorted one: the same lanes take the same edges, products are rounded alike and forces are
summed as integers, so gradient and embedding agree bit for bit."""
import numpy as np
import pytest
import torch

from oracle import c_oracle
from paper_2505_15511_amd import EDGES_EXCHANGED, EDGES_LDS_SUMS, EDGES_POOLED, EDGES_RECORDS, EDGES_ROWS, SCATTER_ATOMIC, Nomad
from tests.test_gpu_parity import GRAD_TOL, grad_err

pytestmark = pytest.mark.gpu
BLOCK = {1: 3072, 2: 3072, 3: 2304, 4: 1536, 5: 1536, 6: 768, 7: 768, 8: 768}     # positions of a block


def graph(n, E, seed, hub=0):
    """E edges with random heads (rows of every length, empty ones too) and tails; with `hub`, that many of them leave one point."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    head = torch.randint(0, n, (E,), generator=g, device="cuda")
    head[:hub] = n // 3
    head = head.sort().values
    col = (head + 1 + torch.randint(0, max(1, n - 1), (E,), generator=g, device="cuda")) % n
    near = torch.rand(E, generator=g, device="cuda") < 0.5                # half of the tails close by: long runs of one tile
    col = torch.where(near, (head + 1 + torch.randint(0, min(40, n - 1), (E,), generator=g, device="cuda")) % n, col)
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(head, minlength=n), 0).to(torch.int32)
    return row_ptr, col.to(torch.int32), 0.5 * torch.randn(n, 2, generator=g, device="cuda")


def epochs(n, s, row_ptr, col, theta, exchange, tune=None, weights=None, n_epochs=2, **kw):
    nm = Nomad(n, 1, s, 5.0, 10, 1.0, 77, tune=dict(tune or {}, exchange=exchange), **kw)
    nm.set_graph(row_ptr, col, weights, torch.zeros(n, dtype=torch.int32, device="cuda"), None)
    assert nm.edge_pass() == (EDGES_EXCHANGED if exchange == 1 else EDGES_RECORDS) and nm.note() == ""
    nm.set_embedding(theta)
    for t in range(n_epochs):
        nm.epoch(t)
    return nm.get_gradient(device=True), nm.get_embedding(device=True)


def same(a, b):
    assert torch.equal(a[0].view(torch.int32), b[0].view(torch.int32)) and torch.equal(a[1].view(torch.int32), b[1].view(torch.int32))


@pytest.mark.parametrize("s", range(1, 9))
@pytest.mark.parametrize("blocks,edges", [(0, 1), (0, 63), (1, -1), (1, 0), (1, 1), (9, 77)])
def test_blocks(s, blocks, edges):
    E = blocks * BLOCK[s] + edges
    args = graph(2_000, E, 100 * s + E % 97, hub=5_000 if blocks == 9 else 0)
    same(epochs(2_000, s, *args, exchange=1), epochs(2_000, s, *args, exchange=2))


@pytest.mark.parametrize("n", [2, 17, 256, 4_097, 65_536, 300_001])
def test_points(n):
    args = graph(n, 40_000, n)
    same(epochs(n, 5, *args, exchange=1), epochs(n, 5, *args, exchange=2))


# tile kernels: 64 lanes a run; 32; pairs of tiles and 32, 16 for the sums; pairs and 16
@pytest.mark.parametrize("n,E", [(1_200_000, 3_000_001), (3_100_000, 3_200_000), (7_000_003, 9_000_000), (17_500_001, 9_000_000)])
def test_lanes_and_pairs(n, E):
    args = graph(n, E, n % 1000, hub=20_000)
    same(epochs(n, 5, *args, exchange=1, n_epochs=1), epochs(n, 5, *args, exchange=2, n_epochs=1))


# runs of about as many references as lanes take of one (64; in the mean 63 and 71), of fewer (53) and of more than twice as many (288)
@pytest.mark.parametrize("n,s,blocks", [(300_000, 5, 90), (1_060_000, 3, 300), (1_060_000, 5, 300), (1_060_000, 8, 300), (500, 5, 40)])
def test_runs_longer_than_lanes(n, s, blocks):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + s)
    E = blocks * BLOCK[s] + 321
    head = torch.randint(0, n, (E,), generator=g, device="cuda").sort().values
    col = ((head + 1 + torch.randint(0, n - 1, (E,), generator=g, device="cuda")) % n).to(torch.int32)   # tails anywhere: all runs alike
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(head, minlength=n), 0).to(torch.int32)
    args = row_ptr, col, 0.5 * torch.randn(n, 2, generator=g, device="cuda")
    same(epochs(n, s, *args, exchange=1, n_epochs=1), epochs(n, s, *args, exchange=2, n_epochs=1))


@pytest.mark.parametrize("tune,kw", [({}, {"batches_per_epoch": 4}), ({"record_phases": 3}, {}), ({"record_phases": 64}, {"batches_per_epoch": 3}),
                                     ({}, {"inverse_rank_weights": True})], ids=["sub-steps", "phases", "both", "ranks"])
def test_steps_and_weights(tune, kw):
    args = graph(30_000, 200_000, 5, hub=3_000)
    same(epochs(30_000, 5, *args, exchange=1, tune=tune, **kw), epochs(30_000, 5, *args, exchange=2, tune=tune, **kw))


@pytest.mark.parametrize("n,s,kw,want", [
    (2_000, 5, {}, EDGES_LDS_SUMS), (10_225, 5, {}, EDGES_RECORDS), (300_000, 5, {}, EDGES_RECORDS), (1_000_000, 5, {}, EDGES_EXCHANGED),
    (1_000_000, 2, {}, EDGES_RECORDS), (1_500_000, 2, {}, EDGES_EXCHANGED), (1_000_000, 5, {"batches_per_epoch": 3}, EDGES_RECORDS),
    (1_000_000, 9, {}, EDGES_ROWS), (1_000_000, 5, {"scatter_mode": SCATTER_ATOMIC}, EDGES_ROWS),
    (1_000_000, 5, {"pool_size": 1024, "pool_block": 4096}, EDGES_POOLED), (1_000_000, 5, {"tune": {"record_sort": 1}}, EDGES_RECORDS)])
def test_which_pass(n, s, kw, want):
    row_ptr, col, _ = graph(n, 3_000_000, n)
    nm = Nomad(n, 1, s, 5.0, 10, 1.0, 77, **kw)
    assert nm.edge_pass() == 0
    nm.set_graph(row_ptr, col, None, torch.zeros(n, dtype=torch.int32, device="cuda"), None)
    assert nm.edge_pass() == want
    nm.close()


def test_against_the_oracle():
    n, s = 5_000, 5
    row_ptr, col, theta = graph(n, 60_000, 9, hub=2_000)
    w = torch.rand(60_000, device="cuda") + 0.1
    got = epochs(n, s, row_ptr, col, theta, exchange=1, weights=w, n_epochs=1)
    O = c_oracle.COracle(row_ptr=row_ptr.cpu().numpy(), col_idx=col.cpu().numpy(), weights=w.cpu().numpy(), cluster_of=np.zeros(n, np.int32), 
                         n=n, n_clusters=1, n_neg=s, noise_count=5.0, n_epochs=10, lr0=1.0, seed=77)
    _, g_ref, _ = O.epoch(theta.cpu().numpy(), 0)
    assert grad_err(got[0].cpu().numpy(), g_ref) < GRAD_TOL


@pytest.mark.parametrize("kw", [{"tune": {"record_phases": 3}}, {"batches_per_epoch": 2}], ids=["phases", "sub-steps"])
def test_recorded_epochs(kw):
    """Every replay of a recorded epoch gives what the eager epochs give, with eager work in between."""
    n, s = 30_000, 5
    row_ptr, col, theta = graph(n, 100_000, 6, hub=3_000)
    want = epochs(n, s, row_ptr, col, theta, exchange=1, **kw)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        tune = dict(kw.get("tune", {}), exchange=1)
        nm = Nomad(n, 1, s, 5.0, 10, 1.0, 77, tune=tune, stream=side.cuda_stream, batches_per_epoch=kw.get("batches_per_epoch", 1))
        nm.set_graph(row_ptr, col, None, torch.zeros(n, dtype=torch.int32, device="cuda"), None)
        nm.set_embedding(theta)
        recorded = torch.cuda.CUDAGraph()
        with torch.cuda.graph(recorded, stream=side):
            nm.epoch(0)
            nm.epoch(1)
        for _ in range(3):
            nm.epoch(2)
            nm.set_embedding(theta)
            recorded.replay()
            side.synchronize()
            same((nm.get_gradient(device=True), nm.get_embedding(device=True)), want)
        nm.close()
