"""The neighbour filter's error bound for products that are summed a chunk of columns at a time (csrc/filter_scale.h), on the CPU:
the kernel's arithmetic in numpy, every addition truncated, against float64."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r'''
#include <stdio.h>
#include <stdlib.h>
#include "filter_scale.h"
int main(int, char** a) { printf("%.17g %.17g\n", nomad_knn::knn_filter_eps(atoi(a[1]), atof(a[2]), atoi(a[3])), nomad_knn::knn_filter_eps(atoi(a[1]), atof(a[2]))); }
'''


@pytest.fixture(scope="module")
def bounds(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("chunks")
    src, exe = tmp / "eps.cpp", str(tmp / "eps")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(src), "-o", exe], check=True)
    return lambda d, M, chunk: [float(x) for x in subprocess.run([exe, str(d), repr(float(M)), str(chunk)], check=True, capture_output=True, text=True).stdout.split()]


def _cut(x):   # float64 -> float32 towards zero: a rounding error of up to 2 u, one-sided
    y = x.astype(np.float32)
    over = np.abs(y.astype(np.float64)) > np.abs(x)
    return np.where(over, np.nextafter(y, np.float32(0)), y).astype(np.float32)


@pytest.mark.parametrize("d", [65, 128, 191, 192, 300, 768])
@pytest.mark.parametrize("kind", ["gaussian", "equal", "first chunk", "same point"])
def test_truncated_sums_stay_inside(bounds, d, kind):
    rng = np.random.default_rng(d)
    q, c = rng.normal(size=(2, 24, d)).astype(np.float32) * np.float32(3.0)
    if kind == "equal":                               # every product of the same sign and size: nothing cancels
        q, c = np.abs(q), np.abs(c)
    elif kind == "first chunk":
        q[:, 64:] *= np.float32(1e-3)
        c[:, 64:] *= np.float32(1e-3)
    elif kind == "same point":
        c = (q * (1 + 1e-3 * rng.normal(size=q.shape))).astype(np.float32)
    qd, cd = q.astype(np.float64), c.astype(np.float64)
    M = max((qd ** 2).sum(1).max(), (cd ** 2).sum(1).max())
    def hi(x):
        return x.astype(np.float16)
    qh, ch = hi(q), hi(c)
    ql, cl = hi(q - qh.astype(np.float32)), hi(c - ch.astype(np.float32))
    qh, ch, ql, cl = (x.astype(np.float64) for x in (qh, ch, ql, cl))
    big = ((cd ** 2).sum(1)[None] / 2).astype(np.float32).repeat(24, 0)
    small = np.zeros((24, 24), np.float32)
    chunk = None
    for t in range(d):
        p = -qh[:, t, None] * ch[None, :, t]
        if t < 64:
            big = _cut(big.astype(np.float64) + p)
        else:
            if t % 64 == 0:
                big = big if chunk is None else big + chunk
                chunk = np.zeros((24, 24), np.float32)
            chunk = _cut(chunk.astype(np.float64) + p)
        small = _cut(small.astype(np.float64) - ql[:, t, None] * ch[None, :, t])
        small = _cut(small.astype(np.float64) - qh[:, t, None] * cl[None, :, t])
    key = 2.0 * ((big + chunk) + small).astype(np.float64)
    exact = (cd ** 2).sum(1)[None] - 2.0 * qd @ cd.T
    eps, whole = bounds(d, M, 64)
    assert np.abs(key - exact).max() <= eps <= whole


U = 2.0 ** -24


def _split(x):   # float16 parts as the packing makes them (rows scaled to at most 2^14)
    hi = x.astype(np.float16)
    return hi.astype(np.float64), (x - hi.astype(np.float32)).astype(np.float16).astype(np.float64)


def _norm(c):   # k_knn_norms: sixteen lanes, fused multiply-adds, then pairwise
    lanes = np.zeros(16, np.float32)
    for t, v in enumerate(c):
        lanes[t // 4 % 16] = np.float32(np.float64(lanes[t // 4 % 16]) + np.float64(v) ** 2)
    while len(lanes) > 1:
        lanes = lanes[:len(lanes) // 2] + lanes[len(lanes) // 2:]
    return lanes[0]


def _big(norm, products, chunk):   # additions inside a chunk truncated, the chunks' sums joined to nearest; and the joins in float64
    big, exact, part = np.float32(norm) * np.float32(0.5), None, None
    sums = []
    for t, p in enumerate(products):
        if t >= chunk and t % chunk == 0:
            if part is not None:
                sums.append(part)
            part = np.float32(0)
        if t < chunk:
            big = _cut(np.asarray(np.float64(big) + p))[()]
        else:
            part = _cut(np.asarray(np.float64(part) + p))[()]
    if part is not None:
        sums.append(part)
    exact = np.float64(big)
    for x in sums:
        big = np.float32(big + x)
        exact += np.float64(x)
    return big, exact


def _rows(d, kind, chunk, rng):
    """A query and a candidate near the bound, |q|^2 = |c|^2 about 2^27, every product of the large sum positive (c is about -q)."""
    top = np.float32(2.0 ** 13.5)
    if kind == "early":      # one large column a chunk, the others' products just below its last place: truncated, each is lost whole
        x = np.zeros(d, np.float32)
        first = np.arange(0, d, chunk)
        big = np.float16(np.sqrt(2.0 ** 27 / len(first)))
        x[first] = big
        for f in first:      # (the first chunk's sum begins at |c|^2 / 2)
            at = np.float64(big) ** 2 + (2.0 ** 26 if f == 0 else 0.0)
            rest = x[f:f + chunk]
            rest[rest == 0] = np.float16(np.sqrt(2.0 ** (np.floor(np.log2(at)) - 23) * 0.998))
        return x, -x
    x = np.abs(rng.normal(size=d)) + 0.5 if kind == "one sign" else rng.normal(size=d)
    x = (x * (np.float64(top) / np.sqrt((x ** 2).sum()))).astype(np.float32)
    return x, -(x * (1 + 1e-4 * rng.normal(size=d))).astype(np.float32)


@pytest.mark.parametrize("d", [64, 65, 128, 129, 192, 320, 321, 767, 768])
@pytest.mark.parametrize("kind", ["one sign", "early", "any sign"])
def test_every_term_inside_its_own_allowance(bounds, d, kind):
    """The terms of knn_filter_eps one by one (before doubling: half of what the key is allowed), for whole chunks and one column more."""
    chunk, rng = 64, np.random.default_rng(d)
    q, c = _rows(d, kind, chunk, rng)
    qd, cd = q.astype(np.float64), c.astype(np.float64)
    M = max((qd ** 2).sum(), (cd ** 2).sum())
    (qh, ql), (ch, cl) = _split(q), _split(c)
    norm = _norm(c)
    norm_err = abs(np.float64(norm) - (cd ** 2).sum())
    assert norm_err <= (d / 16 + 10) * U * M
    products = -qh * ch
    big, joined = _big(norm, products, chunk)
    inside = abs(joined - (np.float64(norm) / 2 + products.sum()))
    assert inside <= 3 * (chunk + 1) * U * M
    joins = abs(np.float64(big) - joined)
    assert joins <= 1.5 * (d / chunk + 2) * U * M
    small = np.float32(0)
    for t in range(d):
        small = _cut(np.asarray(np.float64(small) - ql[t] * ch[t]))[()]
        small = _cut(np.asarray(np.float64(small) - qh[t] * cl[t]))[()]
    assert abs(np.float64(small) + (ql * ch + qh * cl).sum()) <= d / 128 * U * M
    assert abs((qd * cd).sum() - (qh * ch + qh * cl + ql * ch).sum()) <= 26 * U * M
    eps, whole = bounds(d, M, chunk)
    key, exact = 2.0 * np.float64(np.float32(big + small)), (cd ** 2).sum() - 2.0 * (qd * cd).sum()
    assert abs(key - exact) <= eps
    print(f"{abs(key - exact) / eps:.2f} of the bound, inside {inside / (3 * (chunk + 1) * U * M):.2f}")
    if kind == "early" and d % chunk == 0:
        assert inside >= 0.5 * 3 * (chunk + 1) * U * M and abs(key - exact) >= 0.4 * eps   # the bound is not much wider than what these rows take
    if kind == "early" and d >= 320:                            # one sum for all columns does not stay inside the chunks' bound
        x, y = _rows(d, kind, d, rng)
        big, _ = _big(_norm(y), -x.astype(np.float64) * y.astype(np.float64), d)
        xd, yd = x.astype(np.float64), y.astype(np.float64)
        assert abs(2.0 * np.float64(big) - ((yd ** 2).sum() - 2.0 * (xd * yd).sum())) > bounds(d, (yd ** 2).sum(), chunk)[0]
