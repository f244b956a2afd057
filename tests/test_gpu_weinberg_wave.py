"""The Weinberg kernel with four cells to a wavefront: counts of cells around
a wave's and a range's remainder, the largest record it takes, and cells with
more candidate walks than lanes."""
import numpy as np
import pytest

import oracle
from paper_2209_11606_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def v():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_11606_amd import vorohip
    return vorohip


def check(v, x, per):
    o = oracle.Oracle(x, [0] * 3, [1] * 3, per)
    r = o.weinberg(nthreads=8)
    g = v.tessellate(torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0"), [0] * 3, [1] * 3, per,
                     v.VC_ALL | v.VC_WEINBERG, cells_per_wave=2)
    codes = v.weinberg_codes(g)
    for i in range(len(x)):
        assert np.array_equal(codes[i], r["codes"][i]), i
        assert g["wb_sym"][i] == r["sym"][i] and g["wb_chiral"][i] == r["chiral"][i], i
    return g


@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 63, 130])
@pytest.mark.parametrize("per", [[1, 1, 1], [0, 0, 0]])
def test_counts(v, n, per):
    check(v, W.uniform(n, 3, 1.0, 300 + n), per)


@pytest.mark.parametrize("shell", [33, 34, 35])
def test_largest_record(v, shell):
    """The cell of a particle in a sphere of `shell` others has that many
    faces: 62, 64 (192 darts, the kernel's limit) and 66 vertices."""
    rng = W.rng(500 + shell)
    u = rng.normal(size=(shell, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    x = np.concatenate([[[0.5, 0.5, 0.5]], 0.5 + 0.1 * u])
    g = check(v, x, [0, 0, 0])
    assert g["nf"][0] == shell and g["nv"][0] == 2 * shell - 4


def test_many_candidates(v):
    """A regular dodecahedron: 120 candidate walks, all of them smallest."""
    t = (1.0 + 5.0 ** 0.5) / 2.0
    u = np.array([(0, a, b * t) for a in (-1, 1) for b in (-1, 1)], float)
    u = np.concatenate([u, u[:, [1, 2, 0]], u[:, [2, 0, 1]]]) / np.sqrt(1.0 + t * t)
    x = np.concatenate([[[0.5, 0.5, 0.5]], 0.5 + 0.1 * u])
    g = check(v, x, [0, 0, 0])
    assert g["nf"][0] == 12 and g["wb_sym"][0] == 120
