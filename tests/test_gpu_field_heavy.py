"""Mean-field sums where one group holds much of the mass and the others are far from it: what a head sums is then a small part of what the field interpolates, and the
error has to stay small against that part.  Sums in float64 are the reference, errors are relative to each head's own sum of magnitudes."""
import pytest
import torch

from paper_2505_15511_amd import Nomad
from tests.test_gpu_exchange import graph
from tests.test_gpu_field import in_float64, spread

pytestmark = pytest.mark.gpu
N, R = 1_000_003, 701


def heavy_group(share, cells, away, corner, seed):
    """A group of `cells` cells with `share` of the points around (-away / 2, 0.2), all others their own groups around (away / 2, -0.1)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    first = int(share * N)
    i = torch.arange(N, device="cuda")
    cluster_of = torch.where(i < first, i * cells // first, cells + (i - first) * (R - cells) // (N - first)).to(torch.int32)
    groups = (torch.arange(R, device="cuda") - cells + 1).clamp_(min=0).to(torch.int32)
    th = 0.15 * torch.randn(N, 2, generator=g, device="cuda").clamp_(-4.0, 4.0)
    th[:, 0] += torch.where(i < first, -away / 2, away / 2)
    th[:, 1] += torch.where(i < first, 0.2, -0.1) + (torch.where(i < first, -away / 2, away / 2) if corner else 0.0)
    return th, cluster_of, groups


# by interpolation: rounded once to float32 (2^-24 of the value at most), and as much again is what the rule allows the interpolants; cell by cell in float32: some twenty
# roundings of terms and partial sums at most, in any direction
@pytest.mark.parametrize("share,cells,away,corner,field", [
    (0.05, 1, 8.0, False, True), (0.1, 1, 25.0, False, True), (0.5, 1, 5.0, False, True), (0.5, 7, 10.0, False, True), (0.5, 1, 20.0, False, True),
    (0.9, 1, 10.0, False, True), (0.5, 1, 50.0, True, False), (0.9, 7, 25.0, False, False), (0.99, 1, 20.0, False, False), (0.9999, 1, 10.0, False, False)])
def test_errors_are_relative_to_what_is_summed(share, cells, away, corner, field):
    th, cluster_of, groups = heavy_group(share, cells, away, corner, int(away))
    nm = Nomad(N, R, 2, 5.0, 10, 1.0, 5)
    row_ptr, col, _ = graph(N, 60_000, 7)
    nm.set_graph(row_ptr, col, None, cluster_of, groups)
    nm.set_embedding(th)
    heads = torch.cat([torch.arange(2_000), torch.arange(N - 60, N), torch.randint(0, N, (1_000,), generator=torch.Generator().manual_seed(3))]).cuda()
    mu, counts = (torch.as_tensor(v).cuda() for v in nm.get_means())
    A, B = (torch.as_tensor(v).cuda()[heads].double() for v in nm.get_mean_field())
    of, gr = cluster_of.long(), groups.long()
    wantA, wantB = in_float64(th, mu, counts, of, gr, heads)
    d = th[heads].double()[:, None, :] - mu.double()[None]
    q = 1.0 / (1.0 + (d ** 2).sum(-1))
    p = (counts.double() / N).float().double() * (gr[of[heads]][:, None] != gr[None])
    sizeB = (p * q * q * d.norm(dim=-1)).sum(1)
    tol = 2.0 ** -23 if field else 2e-6
    assert ((A - wantA).abs() <= tol * wantA).all(), float(((A - wantA).abs() / wantA).max())
    assert ((B - wantB).norm(dim=1) <= tol * 2 ** 0.5 * sizeB).all(), float(((B - wantB).norm(dim=1) / sizeB).max())
    nm.close()


def test_sub_steps_over_many_squares():
    """Only points of the second half have edges: the second of two sub-steps, whose heads they are, has the gradient of one step over all heads."""
    n, cells, E = 600_001, 4_000, 60_000
    g = torch.Generator(device="cuda").manual_seed(1)
    head = (n // 2 + torch.randint(0, n - n // 2, (E,), generator=g, device="cuda")).sort().values
    col = ((head + 1 + torch.randint(0, n - 1, (E,), generator=g, device="cuda")) % n).to(torch.int32)
    row_ptr = torch.zeros(n + 1, dtype=torch.int32, device="cuda")
    row_ptr[1:] = torch.cumsum(torch.bincount(head, minlength=n), 0).to(torch.int32)
    cluster_of = (torch.arange(n, device="cuda") * cells // n).to(torch.int32)
    th = spread(n, cluster_of.long(), cells, "clusters", 7)
    got = []
    for batches in (1, 2):
        nm = Nomad(n, cells, 2, 5.0, 10, 0.0, 5, batches_per_epoch=batches)
        nm.set_graph(row_ptr, col, None, cluster_of, torch.arange(cells, dtype=torch.int32, device="cuda"))
        nm.set_embedding(th)
        nm.epoch(0)
        got.append(nm.get_gradient(device=True))
        nm.close()
    assert (got[0] - got[1]).abs().max() <= 2.0 ** -21 * got[0].abs().max()


@pytest.mark.parametrize("size", [1e-4, 1e-3, 1e-2])
def test_a_small_embedding_off_the_centre_of_its_square(size):
    """Heads and cells so close that every B is a difference of nearby points: as exact as the sums cell by cell."""
    n, cells = 1_000_003, 600
    g = torch.Generator(device="cuda").manual_seed(4)
    cluster_of = (torch.arange(n, device="cuda") * cells // n).to(torch.int32)
    groups = torch.arange(cells, device="cuda")
    th = size * (torch.randn(n, 2, generator=g, device="cuda") + torch.randn(cells, 2, generator=g, device="cuda")[cluster_of.long()]) + torch.tensor([0.21, 2.9], device="cuda")
    nm = Nomad(n, cells, 2, 5.0, 10, 1.0, 5)
    row_ptr, col, _ = graph(n, 60_000, 7)
    nm.set_graph(row_ptr, col, None, cluster_of, groups.to(torch.int32))
    nm.set_embedding(th)
    heads = torch.randint(0, n, (3_000,), generator=torch.Generator().manual_seed(3)).cuda()
    mu, counts = (torch.as_tensor(v).cuda() for v in nm.get_means())
    B = torch.as_tensor(nm.get_mean_field()[1]).cuda()[heads].double()
    _, wantB = in_float64(th, mu, counts, cluster_of.long(), groups, heads)
    d = th[heads].double()[:, None, :] - mu.double()[None]
    p = (counts.double() / n).float().double() * (cluster_of.long()[heads][:, None] != groups[None])
    sizeB = (p * d.norm(dim=-1) / (1.0 + (d ** 2).sum(-1)) ** 2).sum(1)
    assert ((B - wantB).norm(dim=1) <= 2.0 ** -23 * 2 ** 0.5 * sizeB).all(), float(((B - wantB).norm(dim=1) / sizeB).max())
    nm.close()
