"""The side predicate of the 2D cell kernels on the host, against exact
rationals: the sign of
    s * D(a,b) = -h_a D(b,p) + h_b D(a,p) - h_p D(a,b)
for the vertex of lines a and b and a line p (bisectors, radical lines of
section 2.1.1, walls), by the expansions and by the double-word stage in front
of them, which must decide every sign but an exact zero's."""
import os
import random
import shutil
import subprocess
from fractions import Fraction as F

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HEADER = os.path.join(HERE, "..", "paper_2209_11606_amd", "csrc", "cell_common.h")

HARNESS = r"""
#include <cstdio>
#include <cmath>
#define __device__
#define __noinline__
#define __forceinline__ inline
using std::fabs;
%s
static double ws[kXsLen];
template <class P>
static void run(P *pl) {
    const P *r[3] = {&pl[0], &pl[1], &pl[2]};
    double nv[3][2];
    for (int i = 0; i < 3; i++) {
        nv[i][0] = plane_base(pl[i]).n0;
        nv[i][1] = plane_base(pl[i]).n1;
    }
    const int quick = dw_side2<P>(r, nv);
    printf("%%d %%d\n", exact_side2(pl[0], pl[1], pl[2], ws), quick);
}
int main() {
    int rad;
    double ri;
    while (scanf("%%d %%la", &rad, &ri) == 2) {
        PlaneD d[3];
        PlaneR q[3];
        for (int i = 0; i < 3; i++) {
            double n0, n1, h, rj;
            int wall;
            if (scanf("%%la %%la %%d %%la %%la", &n0, &n1, &wall, &h, &rj) != 5) return 1;
            d[i] = PlaneD{n0, n1, 0.0, h, wall};
            q[i] = PlaneR{d[i], ri, rj};
        }
        if (rad) run(q); else run(d);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def predicate(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    src = open(HEADER).read()
    a, b = src.index("struct PlaneD {"), src.index("// r_i^2 - r_j^2 of a radical plane")
    d = tmp_path_factory.mktemp("pred2")
    cpp, exe = d / "pred.cpp", d / "pred"
    cpp.write_text(HARNESS % src[a:b])
    subprocess.run([gxx, "-O2", "-std=c++17", "-ffp-contract=off", "-o", str(exe), str(cpp)], check=True)

    def call(cases):
        lines = []
        for rad, ri, planes in cases:
            toks = [str(int(rad)), float(ri).hex()]
            for n, wall, h, rj in planes:
                toks += [float(n[0]).hex(), float(n[1]).hex(), str(int(wall)), float(h).hex(), float(rj).hex()]
            lines.append(" ".join(toks))
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        return [tuple(map(int, l.split())) for l in out.stdout.split("\n") if l.strip()]
    return call


def exact_sign(rad, ri, planes):
    n = [[F(float(x)) for x in p[0]] for p in planes]
    h = []
    for nf, (_, wall, hw, rj) in zip(n, planes):
        v = sum(x * x for x in nf) + (F(float(ri)) ** 2 - F(float(rj)) ** 2 if rad else 0)
        h.append(F(float(hw)) if wall else v / 2)

    def det(i, j):
        return n[i][0] * n[j][1] - n[i][1] * n[j][0]
    num = -h[0] * det(1, 2) + h[1] * det(0, 2) - h[2] * det(0, 1)
    den = det(0, 1)
    return ((num > 0) - (num < 0)) * ((den > 0) - (den < 0))


def near_tie(rng, scale, rel):
    """Two random bisectors and a third through their vertex up to rounding,
    optionally moved by a relative amount."""
    q = rng.normal(size=(2, 2)) * scale
    v = np.linalg.solve(q, 0.5 * (q * q).sum(1))
    t = rng.uniform(0, 2 * np.pi)
    p = (v + np.linalg.norm(v) * np.array([np.cos(t), np.sin(t)])) * (1.0 + rel)
    return [(row, 0, 0.0, 0.0) for row in np.vstack([q, p])]


def lattice(rng):
    while True:
        q = rng.integers(-3, 4, size=(3, 2)).astype(float)
        if np.all(np.any(q != 0, 1)):
            return q


def check(cases, got):
    zeros = 0
    for (rad, ri, planes), (full, quick) in zip(cases, got):
        want = exact_sign(rad, ri, planes)
        assert full == want
        assert quick == (2 if want == 0 else want)
        zeros += want == 0
    return zeros


def test_voronoi_near_and_exact_ties(predicate):
    rng = np.random.default_rng(21)
    cases = []
    for t in range(1500):
        if t % 3 == 0:
            planes = near_tie(rng, 10.0 ** rng.uniform(-3, 3), 0.0)
        elif t % 3 == 1:
            planes = near_tie(rng, 1.0, rng.choice([-1, 1]) * 10.0 ** rng.uniform(-15, -6))
        else:
            planes = [(row, 0, 0.0, 0.0) for row in lattice(rng)]
        cases.append((False, 0.0, planes))
    assert check(cases, predicate(cases)) > 50


def test_walls_and_radical_lines(predicate):
    rng = np.random.default_rng(22)
    cases = []
    for t in range(900):
        planes = near_tie(rng, 1.0, 0.0 if t % 2 else 10.0 ** rng.uniform(-14, -7))
        if t % 3 == 0:
            nrm = np.zeros(2)
            nrm[int(rng.integers(2))] = rng.choice([-1.0, 1.0])
            planes[int(rng.integers(3))] = (nrm, 1, float(rng.uniform(0.1, 2.0)), 0.0)
        rad = t % 3 == 1
        ri = float(rng.uniform(0.0, 0.3)) if rad else 0.0
        if rad:
            planes = [(n, w, h, float(rng.uniform(0.0, 0.3))) for n, w, h, _ in planes]
        cases.append((rad, ri, planes))
    for t in range(100):
        cases.append((True, 0.25, [(row, 0, 0.0, 0.25) for row in lattice(rng)]))
    assert check(cases, predicate(cases)) > 5


def test_scaled_lattices_one_ulp_off(predicate):
    rng, r = np.random.default_rng(23), random.Random(23)
    cases = []
    for t in range(300):
        q = lattice(rng) * 2.0 ** r.randint(-40, 40)
        if t % 2:
            i = r.randrange(3)
            d = r.choice(np.flatnonzero(q[i]).tolist())  # (beside zero lies a denormal, whose products underflow)
            q[i][d] = np.nextafter(q[i][d], np.inf)
        cases.append((False, 0.0, [(row, 0, 0.0, 0.0) for row in q]))
    for case, (full, _) in zip(cases, predicate(cases)):
        assert full == exact_sign(*case)
