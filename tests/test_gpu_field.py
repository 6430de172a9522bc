"""Mean-field sums by interpolation against the sums in float64, over the squares' edges, embeddings that the field cannot use, groups of several cells, sub-steps and
recorded epochs."""
import pytest
import torch

from paper_2505_15511_amd import Nomad
from tests.test_gpu_exchange import graph

pytestmark = pytest.mark.gpu


def problem(n, R, cells_per_group=1, **kw):
    row_ptr, col, _ = graph(n, 60_000, n % 89)
    cluster_of = (torch.arange(n, device="cuda") * R // n).to(torch.int32)
    groups = (torch.arange(R, dtype=torch.int32, device="cuda") // cells_per_group)
    nm = Nomad(n, R, 2, 5.0, 10, 1.0, 5, **kw)
    nm.set_graph(row_ptr, col, None, cluster_of, groups)
    return nm, cluster_of.long(), groups.long()


def spread(n, cluster_of, R, kind, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    th = torch.randn(n, 2, generator=g, device="cuda")
    if kind == "tight":
        return 0.01 * th
    if kind == "clusters":       # within 6 of the origin: at most 169 squares, where the field pays up to 370 (250,003 x 2,100: 4,096 squares R + 1,100 n <= 6.566 n R)
        return 0.5 * th.clamp_(-3.0, 3.0) + 1.2 * torch.randn(R, 2, generator=g, device="cuda").clamp_(-3.5, 3.5)[cluster_of]
    if kind == "edges":          # on the edges and corners of squares, and next to them
        return torch.round(2.0 * th) / 2.0 + 1e-7 * torch.randint(-1, 2, (n, 2), generator=g, device="cuda")
    if kind == "far off":        # near the squares' outer edge
        return 0.1 * th + torch.tensor([30.0, -30.2], device="cuda")
    th = 0.5 * th
    th[n // 3] = torch.tensor([40.0, 1.0], device="cuda") if kind == "outside" else torch.tensor([31.0, -31.0], device="cuda")
    return th


def in_float64(th, mu, counts, cluster_of, groups, heads):
    n = th.shape[0]
    p = (counts.double() / n).float().double()
    d = th[heads].double()[:, None, :] - mu.double()[None]
    q = 1.0 / (1.0 + (d ** 2).sum(-1))
    w = p * q * (groups[cluster_of[heads]][:, None] != groups[None])
    return w.sum(1), ((w * q)[..., None] * d).sum(1)


@pytest.mark.parametrize("kind", ["tight", "clusters", "edges", "far off", "outside", "at the edge"])
@pytest.mark.parametrize("n,R,per", [(250_003, 2_100, 1), (1_000_001, 600, 20)])
def test_sums(n, R, per, kind):
    nm, cluster_of, groups = problem(n, R, per)
    th = spread(n, cluster_of, R, kind, R)
    nm.set_embedding(th)
    heads = torch.cat([torch.arange(300), torch.arange(n - 300, n), torch.randint(0, n, (1_500,)), torch.tensor([n // 3])]).cuda()
    for _ in range(2):                                  # a second time on what the first has left
        mu, counts = (torch.as_tensor(v).cuda() for v in nm.get_means())
        A, B = (torch.as_tensor(v).cuda()[heads].double() for v in nm.get_mean_field())
        wantA, wantB = in_float64(th, mu, counts, cluster_of, groups, heads)
        if kind in ("outside", "at the edge"):           # cell by cell in float32
            assert (A - wantA).abs().max() <= 2e-6 * wantA.max() and (B - wantB).abs().max() <= 2e-6 * wantB.abs().max()
        else:       # one rounding to float32 (2^-24 of the value), the interpolants' 4e-10 and 2e-9 of the cells' mass, which is 1
            assert ((A - wantA).abs() <= 2.0 ** -24 * wantA + 4e-10).all(), float(((A - wantA).abs() / wantA).max())
            assert ((B - wantB).abs() <= 2.0 ** -24 * wantB.abs() + 2e-9).all()


def test_sub_steps_epochs_and_recorded_epochs_agree():
    n, R = 300_007, 4_000
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        nm, cluster_of, _ = problem(n, R, batches_per_epoch=2, stream=side.cuda_stream)
        for kind in ("tight", "clusters", "outside"):
            theta0 = spread(n, cluster_of, R, kind, 7)
            nm.set_embedding(theta0)
            for t in range(3):
                nm.epoch(t)
            side.synchronize()
            want = nm.get_embedding(device=True), nm.get_gradient(device=True)
            recorded = torch.cuda.CUDAGraph()
            nm.set_embedding(theta0)
            with torch.cuda.graph(recorded, stream=side):
                for t in range(3):
                    nm.epoch(t)
            for replay in range(3):
                nm.set_embedding(theta0)
                if replay == 1:
                    nm.loss(2)
                    nm.epoch(1)
                    nm.set_embedding(theta0)
                recorded.replay()
                side.synchronize()
                assert torch.equal(nm.get_embedding(device=True), want[0]) and torch.equal(nm.get_gradient(device=True), want[1]), (kind, replay)
        nm.close()
