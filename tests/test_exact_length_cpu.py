"""The floating-point expansions of the exact side predicate on the host: an
accumulator never holds more components than its workspace has places, and its
sign is the exact sum's (against Python fractions).

The sums spread single bits over the whole range of the doubles, which is what
the longest nonoverlapping expansions look like; products beyond that range
(infinities and NaN, whose sign is not defined) must not write past the end
either."""
import os
import random
import re
import shutil
import subprocess
from fractions import Fraction as F

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
static double ws[8192];
int main() {
    int m;
    while (scanf("%%d", &m) == 1) {
        const double mark = 0x1.5p+7;
        for (double &x : ws) x = mark;
        int n = 0, most = 0, past = 0;
        for (int k = 0; k < m; k++) {
            double a, b;
            if (scanf("%%la %%la", &a, &b) != 2) return 1;
            n = xs_add_prod(ws, n, a, b);
            if (n > most) most = n;
        }
        for (int k = %d; k < 8192; k++) past += !(ws[k] == mark);
        printf("%%d %%d %%d\n", most, past, n ? xs_sign(ws, n) : 0);
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def accumulate(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    internal = open(os.path.join(os.path.dirname(HEADER), "vc_internal.h")).read()
    places = int(re.search(r"kExactDoubles = (\d+);", internal).group(1))
    src = open(HEADER).read()
    a, b = src.index("struct PlaneD {"), src.index("// Exact sign of n_p.v - h_p at the 2D vertex")
    d = tmp_path_factory.mktemp("len")
    cpp, exe = d / "len.cpp", d / "len"
    cpp.write_text(HARNESS % (src[a:b], places))
    subprocess.run([gxx, "-O2", "-std=c++17", "-ffp-contract=off", "-o", str(exe), str(cpp)], check=True)

    def call(sums):
        lines = [str(len(s)) + " " + " ".join(x.hex() for p in s for x in p) for s in sums]
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        return [tuple(map(int, l.split())) for l in out.stdout.split("\n") if l.strip()]
    return call


def bit(r, lo, hi):
    return r.choice([-1.0, 1.0]) * 2.0 ** r.randint(lo, hi)


def test_components_of_finite_sums(accumulate):
    r = random.Random(17)
    sums = []
    for t in range(400):
        m = r.randint(1, 400)
        # products within the doubles' range and exact there: down to 2^-1074
        if t % 3 == 0:
            s = [(bit(r, -537, 510), bit(r, -537, 510)) for _ in range(m)]
        elif t % 3 == 1:
            s = [(r.uniform(-1, 1) * 2.0 ** r.randint(-450, 500), r.uniform(-1, 1) * 2.0 ** r.randint(-450, 500))
                 for _ in range(m)]
        else:
            # one bit every 53 or more places, and the same again with some
            # taken back: as many components as there can be
            e = list(range(1020, -1075, -r.choice([53, 54, 55])))
            s = [(r.choice([-1.0, 1.0]), 2.0 ** k) for k in e]
            s += [(-a, b) for a, b in r.sample(s, len(s) // 2)] + [(bit(r, -537, 500), bit(r, -537, 500)) for _ in range(20)]
            r.shuffle(s)
        sums.append(s)
    for s, (most, past, sign) in zip(sums, accumulate(sums)):
        v = sum(F(a) * F(b) for a, b in s)
        assert past == 0 and most <= 40
        assert sign == (v > 0) - (v < 0)


def test_components_beyond_the_range(accumulate):
    r = random.Random(18)
    sums = [[(bit(r, -900, 900) * r.uniform(1, 2), bit(r, 0, 900) * r.uniform(1, 2)) for _ in range(400)] for _ in range(200)]
    assert all(past == 0 for _, past, _ in accumulate(sums))
