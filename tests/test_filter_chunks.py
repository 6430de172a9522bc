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
