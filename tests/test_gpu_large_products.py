"""Lloyd's iterations whose filter multiplies the high halves alone where these decide for nearly all points: labels, centroids and iterations are the
oracle's, bit for bit, in every instance of that filter and where calls go over to it and back.

Which steps take it is followed here, from the bound of csrc/knn_filter_kernel.h and the rules of csrc/kmeans_plan.h: the points are such that the share
of open ones is far from the rule's line on either side, whatever sample it is taken from."""
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import kmeans_oracle as km
from paper_2505_15511_amd import kmeans_lloyd

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "kmeans_plan.h"
using namespace nomad_knn;
int main(int, char** a) {   // n K d tiles steps M
    const long long n = atoll(a[1]), K = atoll(a[2]), d = atoll(a[3]);
    long long open = 0;
    while (products_alone(open + 64, n, K, d)) open += 64;
    printf("%d %lld %.17g\n", (int)products_may_be_alone(n, K, d, atoll(a[4]), atoll(a[5]), d % 4 == 0), open, knn_filter_eps((int)d, atof(a[6])));
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    t = tmp_path_factory.mktemp("alone")
    (t / "rules.cpp").write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(t / "rules.cpp"), "-o", str(t / "rules")], check=True)

    def ask(n, K, d, steps, M):
        out = subprocess.run([str(t / "rules")] + [repr(x) for x in (n, K, d, -(-n // (32 if d <= 256 else 16)), steps, float(M))], check=True, capture_output=True, text=True).stdout.split()
        return bool(int(out[0])), int(out[1]), float(out[2])
    return ask


def _assign(X, C):
    """The oracle's E step on the GPU, float64, the same operations in the same order: labels, and the two least distances."""
    Cd = torch.from_numpy(C).cuda().double()
    labels, least = [], []
    for rows in torch.split(X, max(1, 60_000_000 // len(C))):
        rows = rows.double()
        D = torch.zeros(len(rows), len(C), dtype=torch.float64, device="cuda")
        for t in range(X.shape[1]):
            e = rows[:, t][:, None] - Cd[None, :, t]
            D += e * e
        labels.append(D.argmin(1))
        least.append(torch.topk(D, 2, dim=1, largest=False).values)
        tie = least[-1][:, 0] == least[-1][:, 1]
        if tie.any():                                            # the first of equal ones
            labels[-1][tie] = (D[tie] == least[-1][tie, :1]).to(torch.int8).argmax(1)
    return torch.cat(labels).cpu().numpy(), torch.cat(least)


def _run(rules, X, C0, iters):
    """Labels, centroids, iterations, and per step the share of the points that the large products leave open over the most they may."""
    n, d = X.shape
    Xg = torch.from_numpy(X).cuda()
    mean = Xg.double().mean(0)                                   # (the filter's centre is a sample's mean: the same to a few parts in a hundred of the lengths)
    length = (Xg.double() - mean).norm(dim=1)
    C, labels, shares = C0, None, []
    for it in range(1, iters + 1):
        new, least = _assign(Xg, C)
        longest = float((torch.from_numpy(C).cuda().double() - mean).norm(dim=1).max())
        may, most, eps = rules(n, len(C), d, iters, max(float(length.max()), longest) ** 2)
        assert may
        slack = 2.0 * 2.02 * 2.0 ** -11 * length * longest       # |hi lo + lo hi|, in the squared distance
        gap = least[:, 1] - least[:, 0]
        shares.append([float((gap <= f * (2 * eps + 2 * slack)).sum()) / most for f in (0.8, 1.25)])
        if labels is not None and np.array_equal(new, labels):
            return C, labels, it, shares
        labels, C = new, km.update(X, new, C)
    return C, labels, iters, shares


def _alone(shares):
    """Per step after the first: whether it takes the large products alone (None: too near the line to tell)."""
    return [True if hi < 0.6 else False if lo > 1.7 else None for lo, hi in shares[:-1]]


def _blobs(n, d, K, rng, spread=0.02):
    centres = rng.normal(size=(K, d)).astype(np.float64)
    c = rng.integers(0, K, n)
    return centres, c, centres[c] + spread * rng.normal(size=(n, d))


# 32- and 16-row tiles, every number of steps once; centroids that don't fill their last tile; rows that are not read 16 bytes at a time
INSTANCES = [(112000, 16, 600), (112000, 31, 601), (33000, 64, 521), (33001, 92, 400), (32800, 128, 300), (33000, 192, 200), (32768, 252, 199), (36000, 300, 100), (34000, 500, 65),
             (22001, 764, 64), (66000, 301, 1025), (131072, 67, 520)]


@pytest.mark.parametrize("n,d,K", INSTANCES)
def test_every_instance(rules, n, d, K):
    """Blobs with a centroid each, and one of half as many points as may be open with two that are alike: these points are open in every step."""
    rng = np.random.default_rng(n + d)
    centres, c, X = _blobs(n, d, K - 1, rng)
    _, most, _ = rules(n, K, d, 4, 1.0)
    few = rng.choice(n, most // 3, replace=False)
    X[c == 0] = (X - centres[0] + centres[1])[c == 0]            # blob 0 is those few
    X[few] = centres[0] + 0.02 * rng.normal(size=(len(few), d))
    X = X.astype(np.float32)
    C0 = np.concatenate([centres, centres[:1] + 1e-4 * rng.normal(size=(1, d))]).astype(np.float32)
    for iters in (2, 4):
        ref = _run(rules, X, C0, iters)
        assert ref[2] == iters and all(_alone(ref[3])) and ref[3][-1][0] > 0.1        # every step from the second on, with points for the refinement
        _same(X, C0, iters, ref)


def _beside_blobs(n, d, K, rng):
    """K - 2 blobs with a centroid each, a quarter of the points for a blob of another shape, and a direction."""
    centres, c, X = _blobs(n, d, K - 2, rng)
    u = rng.normal(size=d)
    return centres, X, rng.random(n) < 0.25, u / np.linalg.norm(u), np.sqrt(d)


def _same(X, C0, iters, ref):
    C_ref, lab_ref, it_ref, _ = ref
    C, lab, it, _ = kmeans_lloyd(torch.from_numpy(X).cuda(), torch.from_numpy(C0.copy()).cuda(), iters)
    assert it == it_ref and np.array_equal(lab.cpu().numpy().astype(np.int64), lab_ref)
    assert np.array_equal(C.cpu().numpy(), C_ref)


@pytest.mark.parametrize("n,d,K", [(33000, 128, 300), (34000, 320, 120)])
def test_to_all_products(rules, n, d, K):
    """A blob, thin along the line through two far centroids, which come to it: few of its points are open at first, all of them in the step after."""
    rng = np.random.default_rng(n)
    centres, X, blob, u, far = _beside_blobs(n, d, K, rng)
    at = rng.normal(size=d)
    flat = 0.02 * rng.normal(size=(n, d))
    X[blob] = (at + flat + ((0.02 * far * rng.normal(size=n)) - flat @ u)[:, None] * u)[blob]
    X = X.astype(np.float32)
    C0 = np.concatenate([(at + far * u)[None], (at - far * u)[None], centres]).astype(np.float32)
    ref = _run(rules, X, C0, 4)
    assert _alone(ref[3])[:2] == [True, False], ref[3]
    _same(X, C0, 4, ref)


@pytest.mark.parametrize("n,d,K", [(33000, 128, 300), (34000, 320, 120)])
def test_from_all_products(rules, n, d, K):
    """A long blob with two centroids that are alike: all of its points are open at first, few once these have parted."""
    rng = np.random.default_rng(n + 1)
    centres, X, blob, u, far = _beside_blobs(n, d, K, rng)
    X[blob] = (0.02 * rng.normal(size=(n, d)) + (far * rng.random(n) ** 3)[:, None] * u)[blob]
    X = X.astype(np.float32)
    C0 = np.concatenate([(0.2 * far + 1e-4) * u[None], 0.2 * far * u[None], centres]).astype(np.float32)
    ref = _run(rules, X, C0, 4)
    assert _alone(ref[3])[0] is False and _alone(ref[3])[1:].count(True) >= 1, ref[3]
    _same(X, C0, 4, ref)


def _case(kind, n, d, K, rng):
    centres = (30.0 if kind == "tight" else 4.0) * rng.normal(size=(K // 4, d))
    X = centres[rng.integers(0, K // 4, n)] + (1e-2 if kind == "tight" else 1.0) * rng.normal(size=(n, d))   # tight: all of a cluster's points and centroids alike to float16
    if kind == "tails":
        X *= np.exp(rng.normal(size=(n, 1)))
    if kind == "grid":
        X = rng.integers(0, 3, (n, d))
    X = X.astype(np.float32)
    C0 = X[rng.choice(n, K, replace=False)].copy()
    if kind == "spread":                                    # far off at first: the centroids come in by and by
        C0 = (8.0 * C0).astype(np.float32)
    return X, C0


# rows that leave most points open, some or none, at sizes that may take it and that may not
@pytest.mark.parametrize("kind,n,d,K", [
    ("plain", 66000, 16, 40), ("plain", 65537, 31, 33), ("plain", 66000, 64, 256), ("plain", 65540, 90, 20), ("plain", 66001, 128, 160), ("spread", 66000, 190, 90),
    ("plain", 65536, 250, 80), ("plain", 65600, 300, 80), ("spread", 65600, 500, 45), ("plain", 65600, 765, 24), ("tight", 66000, 40, 500), ("tight", 65536, 300, 80),
    ("tails", 66000, 24, 700), ("grid", 66000, 5, 30), ("plain", 65535, 20, 16), ("spread", 70000, 9, 50)])
def test_what_the_large_products_decide(kind, n, d, K):
    X, C0 = _case(kind, n, d, K, np.random.default_rng(n + d))
    for iters in (2, 4):
        C_ref, lab_ref, it_ref = C0, None, 0
        while it_ref < iters:
            new, _ = _assign(torch.from_numpy(X).cuda(), C_ref)
            it_ref += 1
            if lab_ref is not None and np.array_equal(new, lab_ref):
                break
            lab_ref, C_ref = new, km.update(X, new, C_ref)
        _same(X, C0, iters, (C_ref, lab_ref, it_ref, None))
