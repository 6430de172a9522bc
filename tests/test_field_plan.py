"""When the mean-field sums may be interpolated (csrc/edge_plan.h, compiled on the host): the error that the rule counts on is what the interpolants have, and where the
rule lets them be used a head's sum without its own group is as exact as float32."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include "edge_plan.h"
using namespace nomad;
// argv: pairs of heaviest, diameter
int main(int argc, char** argv) {
    printf("%.17g %.17g\n", kFieldEdge, kFieldError);
    for (int i = 1; i + 1 < argc; i += 2) printf("%d\n", (int)field_sound(atof(argv[i]), atof(argv[i + 1])));
    printf("%d %d %d\n", (int)field_may(1e6, 1000, 1e6, 0.01), (int)field_may(1e6, 1000, 1e6, 1.0), (int)field_may(1e6, 100, 1e6, 0.01));
    return 0;
}
"""


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    d = tmp_path_factory.mktemp("field_plan")
    src, exe = d / "plan.cpp", d / "plan"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Werror", "-I", os.path.join(ROOT, "paper_2505_15511_amd", "csrc"), str(src), "-o", str(exe)],
                   check=True, capture_output=True, text=True)

    def ask(*pairs):
        out = subprocess.run([str(exe)] + [repr(float(v)) for p in pairs for v in p], check=True, capture_output=True, text=True).stdout.split("\n")
        return [float(v) for v in out[0].split()], [int(v) for v in out[1:1 + len(pairs)]], out[1 + len(pairs)]
    return ask


def kernels(x, y, c):
    dx, dy = x - c[0], y - c[1]
    q = 1.0 / (1.0 + dx * dx + dy * dy)
    return q, q * q * dx, q * q * dy


class Interpolant:
    N = 16

    def __init__(self, edge):
        j, self.half = np.arange(self.N), edge / 2
        self.node = np.cos(np.pi * (j + 0.5) / self.N) * self.half
        self.dct = np.where(j[:, None] == 0, 1.0, 2.0) / self.N * np.cos(np.pi * j[:, None] * (j + 0.5) / self.N)

    def __call__(self, values, x, y):   # values [y][x] at the nodes
        T = [np.cos(np.arange(self.N)[:, None] * np.arccos(np.clip(t / self.half, -1, 1))) for t in (x, y)]
        return np.einsum("yp,yx,xp->p", T[1], self.dct @ values @ self.dct.T, T[0])

    def grid(self):
        return np.meshgrid(self.node, self.node)


def points(rng, half, n=400):
    p = rng.uniform(-half, half, (2, n))
    p[:, : n // 10] = np.sign(p[:, : n // 10]) * half
    return p


def test_error_of_the_interpolants(rule):
    (edge, error), _, _ = rule()
    f, rng = Interpolant(edge), np.random.default_rng(1)
    worst = 0.0
    for k in range(300):
        c = rng.uniform(-edge / 2, edge / 2, 2) if k % 3 else rng.uniform(-2.0, 2.0, 2)
        p = points(rng, edge / 2)
        for got, want in zip(kernels(*f.grid(), c), kernels(*p, c)):
            worst = max(worst, np.abs(f(got, *p) - want).max())
    assert 0.3 * error < worst <= error


def test_lines(rule):
    cases = [(0.5, 30.0, 1), (0.5, 32.0, 0), (0.9, 14.0, 1), (0.9, 16.0, 0), (0.1, 63.0, 1), (0.1, 66.0, 0), (1 / 25, 88.0, 1), (0.99, 5.0, 1), (0.99, 9.0, 0), (1.0, 1.0, 0),
             (0.1, float("nan"), 0), (0.1, float("inf"), 0), (0.1, 1e60, 0)]
    _, got, may = rule(*[c[:2] for c in cases])
    assert got == [c[2] for c in cases]
    assert may == "1 0 0"


@pytest.mark.parametrize("heaviest,away", [(0.5, 2.0), (0.5, 10.0), (0.5, 30.5), (0.9, 14.5), (0.1, 60.0), (0.99, 6.0)])
def test_sums_without_a_heavy_group_are_as_exact_as_float32(rule, heaviest, away):
    """The worst the rule lets pass: all others at the far end of the embedding."""
    (edge, _), got, _ = rule((heaviest, away))
    assert got == [1]
    f, rng = Interpolant(edge), np.random.default_rng(int(away))
    for _ in range(60):
        c, far = rng.uniform(-edge / 2, edge / 2, 2), (away - 0.5 * edge) * np.array([np.cos(0.3), np.sin(0.3)])
        p = points(rng, edge / 2)
        at_nodes = [heaviest * u + (1.0 - heaviest) * v for u, v in zip(kernels(*f.grid(), c), kernels(*f.grid(), far))]
        q, bx, by = [(1.0 - heaviest) * v for v in kernels(*p, far)]
        own = [heaviest * v for v in kernels(*p, c)]
        A, Bx, By = [f(v, *p) - o for v, o in zip(at_nodes, own)]
        assert (np.abs(A - q) <= 2.0 ** -24 * q).all()
        assert (np.maximum(np.abs(Bx - bx), np.abs(By - by)) <= 2.0 ** -24 * np.hypot(bx, by)).all()
