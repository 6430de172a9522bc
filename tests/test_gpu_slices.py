"""Neighbourhood preservation over slices of the set, which tell each other how near their candidates are: what a slice passes over on the
others' account has no part in the answer.  Reference: float64 distances of all pairs, ties by index.  The second space differs from the first by so little that most
neighbours are neighbours in both: a neighbour that is lost in either is missed in the count."""
import pytest
import torch

from paper_2505_15511_amd import NomadError, neighbourhood_preservation

pytestmark = pytest.mark.gpu


def _rows(kind, n, d, g):
    if kind == "grid":                                           # ties in bulk
        return torch.randint(0, 3, (n, d), generator=g).float()
    X = torch.randn(n, d, generator=g)
    if kind == "noise":
        return X
    if kind == "duplicates":
        return X[torch.randint(0, n // 50, (n,), generator=g)]
    c = torch.randint(0, 40, (n,), generator=g)
    if kind == "sorted":                                         # rows of a cluster side by side, one cluster of a few rows
        c = torch.sort(c).values
        c[:7] = 40
    X = X + 4.0 * torch.randn(41, d, generator=g)[c]
    if kind == "offset":                                         # far from the origin, next to the clusters' extent
        X = X + 300.0
    if kind == "tails":
        X = X * torch.exp(1.5 * torch.randn(n, 1, generator=g))
    return X


def _neighbours(A, q, k, ties):
    A = A.double()
    out = []
    for s in torch.split(q, max(1, min(512, 40_000_000 // len(A)))):
        D = torch.zeros(len(s), len(A), dtype=torch.float64, device=A.device)
        for t in range(A.shape[1]):
            e = A[s, t][:, None] - A[None, :, t]
            D += e * e
        D[torch.arange(len(s), device=A.device), s] = float("inf")
        D.nan_to_num_(nan=float("inf"), posinf=float("inf"))     # rows that are no numbers come last
        out.append(torch.sort(D, dim=1, stable=True).indices[:, :k] if ties else torch.topk(D, k, dim=1, largest=False).indices)
    return torch.cat(out)


def _common(a, b):
    return int((a[:, :, None] == b[:, None, :]).sum())


def _slices(n, d, m, k):
    """(slices, rows of one, rows of a tile, rounds of the chip), as neighbours_of_queries cuts the set."""
    tile = 32 if d <= (256 if k + 8 <= 24 else 128) else 16
    blocks = -(-m // (8 * tile))
    cost = lambda g: -(-blocks * g // 256) * -(-n // g)
    G = 1
    for g in range(2, min(256 // k, max(1, n // 4096)) + 1):
        G = g if cost(g) < 0.98 * cost(G) else G
    return G, -(-n // G), tile, blocks * G / 256


def _check(kind, n, d, extra, m, k):
    g = torch.Generator().manual_seed(n + d)
    ties = kind in ("grid", "duplicates")
    if kind == "plane":                                          # points of a plane in d columns, almost: the other space is another search
        Y = torch.randn(n, 2, generator=g) * torch.exp(torch.randn(n, 1, generator=g))
        X = Y @ torch.linalg.qr(torch.randn(d, 2, generator=g)).Q.T + 1e-4 * torch.randn(n, d, generator=g) / d ** 0.5
    else:
        X = _rows(kind, n, d, g)
        more = torch.zeros(n, extra) if ties else 0.1 * torch.randn(n, extra, generator=g)
        Y = torch.cat([X, more], 1)
    q = torch.arange(n) if m == 0 else torch.cat([torch.randperm(n, generator=g)[:m - 2], torch.tensor([n - 1, n - 1])])
    X, Y, q = X.contiguous().cuda(), Y.contiguous().cuda(), q.cuda()
    hits = _common(_neighbours(X, q, k, ties), _neighbours(Y, q, k, ties))
    assert hits >= 0.7 * len(q) * k                              # (the test would see most of what is lost)
    assert neighbourhood_preservation(X, Y, k, None if m == 0 else q.to(torch.int32))[0] == hits


# two slices and more, up to eight and beyond; tiles of 32 and 16 rows, short and long lists, eight wavefronts a workgroup and fewer, all points as queries, a row
# repeated; the last two in several rounds of the chip, where the later slices begin with what the earlier ones have found
@pytest.mark.parametrize("kind,n,d,extra,m,k", [
    ("clusters", 30001, 40, 3, 0, 10), ("clusters", 45000, 128, 30, 21760, 15), ("sorted", 45001, 70, 5, 21000, 12), ("offset", 60000, 20, 3, 16384, 20),
    ("tails", 60000, 33, 8, 16000, 7), ("noise", 90000, 20, 3, 10000, 32), ("grid", 45000, 9, 10, 21000, 10), ("duplicates", 45000, 24, 9, 21000, 15),
    ("clusters", 82003, 16, 60, 1024, 30), ("tails", 380003, 10, 3, 300, 15), ("sorted", 130000, 30, 3, 1024, 25), ("noise", 600000, 6, 4, 3000, 10),
    ("plane", 62000, 300, 0, 8192, 15), ("plane", 62000, 130, 0, 8000, 30), ("plane", 45000, 180, 0, 21000, 10), ("clusters", 290000, 6, 3, 17000, 10),
    ("grid", 150001, 7, 10, 40000, 10)])
def test_what_slices_tell_each_other_has_no_part_in_the_answer(kind, n, d, extra, m, k):
    slices, rows, tile, _ = _slices(n, d, m or n, k)
    long_lists = k + 8 > 24
    assert 1 < slices <= 32 and rows >= (8192 if long_lists and tile == 32 else 14336) and rows * tile >= 1280 * 32 * slices   # they share
    _check(kind, n, d, extra, m, k)


# slices that are too short to, and rows too wide
@pytest.mark.parametrize("kind,n,d,extra,m,k", [
    ("clusters", 20011, 40, 3, 1024, 10), ("sorted", 16385, 70, 5, 1100, 12), ("plane", 12001, 257, 0, 1024, 5), ("tails", 20000, 33, 8, 1024, 7),
    ("grid", 15000, 9, 3, 1024, 10), ("clusters", 8200, 130, 3, 0, 30), ("plane", 9000, 300, 0, 1024, 25), ("clusters", 24001, 16, 84, 1025, 1),
    ("clusters", 70001, 48, 3, 2, 5), ("plane", 25000, 700, 0, 600, 10), ("plane", 45000, 200, 0, 20000, 10)])
def test_slices_that_do_not_share(kind, n, d, extra, m, k):
    _check(kind, n, d, extra, m, k)


@pytest.mark.parametrize("scale", [1e-19, 1e-30, 1e17])
def test_lengths_at_the_ends_of_float32(scale):
    g = torch.Generator().manual_seed(5)
    X = scale * _rows("clusters", 30000, 24, g)
    Y = torch.cat([X, scale * 0.1 * torch.randn(30000, 3, generator=g)], 1).contiguous().cuda()
    X = X.cuda()
    q = torch.arange(30000, device="cuda")
    hits = _common(_neighbours(X, q, 8, False), _neighbours(Y, q, 8, False))
    assert neighbourhood_preservation(X, Y, 8, None)[0] == hits


def test_a_query_that_is_no_row():
    X = _rows("clusters", 20000, 30, torch.Generator().manual_seed(1)).cuda()
    q = torch.arange(1024, dtype=torch.int32, device="cuda")
    q[77] = 20000
    with pytest.raises(NomadError):
        neighbourhood_preservation(X, X[:, :3].contiguous(), 10, q)


# a slice with such a row is the exact path's as a whole and tells nothing; the others share what they have
@pytest.mark.parametrize("value", [float("nan"), float("inf"), 3e38, 1e30])
@pytest.mark.parametrize("scale", [1.0, 1e-9])
def test_rows_that_are_no_numbers(value, scale):
    n, d, k = 60000, 20, 10
    g = torch.Generator().manual_seed(2)
    X = scale * _rows("clusters", n, d, g)
    Y = torch.cat([X, scale * 0.1 * torch.randn(n, 3, generator=g)], 1)
    X[5, 3] = value                                              # in the first of four slices
    q = torch.randperm(n, generator=g)[:16000]
    q = q[q != 5].cuda()
    X, Y = X.contiguous().cuda(), Y.contiguous().cuda()
    hits = _common(_neighbours(X, q, k, False), _neighbours(Y, q, k, False))
    assert hits >= 0.7 * len(q) * k
    assert neighbourhood_preservation(X, Y, k, q.to(torch.int32))[0] == hits
