"""The neighbour filter's scales and error bound (csrc/filter_scale.h) over all magnitudes that float32 holds, on the CPU: the
kernels' arithmetic in numpy, with the header compiled by the host compiler."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROGRAM = r'''
#include <stdio.h>
#include <stdlib.h>
#include "filter_scale.h"
using namespace nomad_knn;
int main(int argc, char** argv) {   // pairs of bit patterns (queries, candidates) -> usable, exponents
    for (int a = 1; a + 1 < argc; a += 2) {
        const uint32_t q = strtoul(argv[a], 0, 0), c = strtoul(argv[a + 1], 0, 0);
        const uint32_t top = q > c ? q : c;
        float M;
        memcpy(&M, &top, sizeof(M));
        printf("%d %d %d %.17g\n", (int)knn_filter_usable(q, c), knn_scale_exponent(q), knn_scale_exponent(c), knn_filter_eps(D, (double)M));
    }
}
'''
D = 24


@pytest.fixture(scope="module")
def scales(tmp_path_factory):
    tmp = tmp_path_factory.mktemp("scale")
    src, exe = tmp / "scale.cpp", str(tmp / "scale")
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", f"-DD={D}", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(src), "-o", exe],
                   check=True)

    def ask(pairs):
        out = subprocess.run([exe] + [str(b) for p in pairs for b in p], check=True, capture_output=True, text=True).stdout.split()
        return [(int(u), int(e), int(f), float(g)) for u, e, f, g in zip(out[0::4], out[1::4], out[2::4], out[3::4])]
    return ask


def _bits(M):
    return int(np.float32(M).view(np.uint32))


def _split(x, e):
    y = (x * np.float32(2.0) ** np.float32(e)).astype(np.float32)
    hi = y.astype(np.float16)
    return hi, (y - hi.astype(np.float32)).astype(np.float16)


def _norms(x):
    s = np.zeros(len(x), np.float32)
    for t in range(x.shape[1]):
        s = (s + x[:, t] * x[:, t]).astype(np.float32)
    return s


@pytest.mark.parametrize("bits", [_bits(np.inf), _bits(np.nan), _bits(-np.nan), 0x7F800001, _bits(3e38)])
def test_groups_without_finite_keys_are_not_filtered(scales, bits):
    ordinary = _bits(40.0)
    assert [u for u, *_ in scales([(bits, bits), (bits, ordinary), (ordinary, bits), (ordinary, ordinary)])] == [0, 0, 0, 1]


@pytest.mark.parametrize("eq", range(-24, 20, 2))
def test_keys_of_filtered_groups_are_finite_and_inside_the_bound(scales, eq):
    rng = np.random.default_rng(eq + 100)
    with np.errstate(all="ignore"):
        for ec in range(-24, 20, 2):
            q, c = ((rng.normal(size=(17, D)) * 10.0 ** e).astype(np.float32) for e in (eq, ec))
            nq, nc = _norms(q), _norms(c)
            (usable, sq, sc, eps), = scales([(_bits(nq.max()), _bits(nc.max()))])
            if max(eq, ec) <= 16 and (eq == ec or min(eq, ec) >= -10):
                assert usable                          # whatever data is filtered in earnest still is
            if not usable:
                continue
            qh, ql = _split(q, sq)
            ch, cl = _split(c, sc)
            half = nc * np.float32(np.ldexp(0.5, sq + sc))
            key = half[None] - (qh.astype(np.float64) @ ch.T.astype(np.float64) + qh.astype(np.float64) @ cl.T.astype(np.float64)
                                + ql.astype(np.float64) @ ch.T.astype(np.float64)).astype(np.float32)
            key = key.astype(np.float32) * np.float32(np.ldexp(2.0, -(sq + sc)))
            assert np.isfinite(half).all() and np.isfinite(key).all()
            exact = (c.astype(np.float64) ** 2).sum(1)[None] - 2.0 * q.astype(np.float64) @ c.T.astype(np.float64)
            assert np.abs(key.astype(np.float64) - exact).max() <= eps
