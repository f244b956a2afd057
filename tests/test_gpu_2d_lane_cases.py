"""The 2D kernel with one cell per lane where its cuts are degenerate and where
it shares a set with the eight-lane kernel: lattices whose candidates come in
any order (cuts through vertices that are there, edges of zero length), axes
with fewer blocks than the offset list reaches, and sets it leaves partly or
wholly.  Against the eight-lane kernel (a vertex capacity selects it) on every
cell and the oracle or the closed form.

Which kernel finished the cells shows in the number of cuts: a lane takes its
particles in the order of the blocks, the eight-lane kernel nearest first."""
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


def run(v, x, box, per, radii=None, **opt):
    xt = torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    return v.tessellate(xt, [0, 0], box, per, v.VC_ALL | v.VC_PERIMETER, radii=radii, **opt)


def same(a, b):
    """Volumes and centroids to 1e-12 of the cell, as every form is held to."""
    for k in ("status", "nv", "ne", "nf", "nbr_off", "nbr_ids", "nbr_sh"):
        assert np.array_equal(a[k], b[k]), k
    assert np.max(np.abs(a["vol"] - b["vol"]) / b["vol"]) <= 1e-12
    assert np.max(np.abs(a["cen"] - b["cen"]).max(1) / np.sqrt(b["vol"])) <= 1e-12
    assert np.max(np.abs(a["perim"] - b["perim"]) / b["perim"]) <= 1e-12


@pytest.mark.parametrize("per", [[1, 1], [0, 0], [0, 1]])
@pytest.mark.parametrize("opt", [dict(), dict(precision=1), dict(radii=0.25), dict(force=2), dict(n_opt=1.0)])
def test_square_lattice(v, per, opt):
    """A unit lattice of 288 x 288 in random input order: every coordinate, line
    and vertex is an exact number of halves, so the cells are exactly squares."""
    m, opt = 288, dict(opt)
    g = np.stack(np.meshgrid(np.arange(m), np.arange(m), indexing="ij"), -1).reshape(-1, 2)
    p = W.rng(41).permutation(m * m)
    x = g[p] + 0.5
    rad = opt.pop("radii", None)
    rad = None if rad is None else np.full(m * m, rad)
    a = run(v, x, [m, m], per, rad, **opt)
    assert np.all(a["status"] == 0)
    assert np.all(a["vol"] == 1.0) and np.all(a["cen"] == 0.0) and np.all(a["perim"] == 4.0)
    for k in ("nv", "ne", "nf"):
        assert np.all(a[k] == 4), k
    at = np.empty(m * m, np.int64)
    at[p] = np.arange(m * m)
    lists = np.sort(a["nbr_ids"].reshape(-1, 4), 1)
    want = np.empty((m * m, 4), np.int64)
    for k, (d, s) in enumerate(((0, -1), (0, 1), (1, -1), (1, 1))):
        t = g[p].copy()
        t[:, d] += s
        out = (t[:, d] < 0) | (t[:, d] >= m)
        t[:, d] %= m
        want[:, k] = np.where(out & (per[d] == 0), -(2 * d + (s > 0) + 1), at[t[:, 0] * m + t[:, 1]])
    assert np.array_equal(lists, np.sort(want, 1))
    b = run(v, x, [m, m], per, rad, capacity=16, **opt)
    same(a, b)
    if not {"force", "n_opt"} & set(opt):
        # (one particle a block: the blocks' order is nearest first too)
        assert a["diag"]["cuts"] > b["diag"]["cuts"]


@pytest.mark.parametrize("k", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("short", [0, 1])
def test_few_blocks_on_an_axis(v, k, short):
    """k blocks across a thin periodic box: neighbours one and two periods off."""
    n = 80_000
    side = 5.0 ** 0.5
    box, grid = [0.0, 0.0], [0, 0]
    box[short], grid[short] = k * side, k
    box[1 - short] = n / box[short]
    grid[1 - short] = int(round(box[1 - short] / side))
    x = W.rng(50 + k).random((n, 2)) * box
    x = np.minimum(x, np.nextafter(box, 0.0))
    a = run(v, x, box, [1, 1], grid=grid)
    b = run(v, x, box, [1, 1], grid=grid, capacity=16)
    same(a, b)
    assert a["diag"]["cuts"] > 1.1 * b["diag"]["cuts"]
    idx = np.arange(0, n, 499)
    r = oracle.Oracle(x, [0, 0], box, [1, 1], grid=grid).cells(idx, nthreads=oracle.num_threads())
    assert np.array_equal(a["nf"][idx], r["nf"])
    assert np.max(np.abs(a["vol"][idx] - r["vol"]) / r["vol"]) <= 1e-12


def test_dense_blocks_are_left(v):
    """1,000 particles a block: every cell goes to the eight-lane kernel; half of
    the set in one small disc: some do."""
    n = 80_000
    x = W.uniform(n, 2, 1.0, 61)
    a, b = run(v, x, [1, 1], [1, 1], grid=[40, 2]), run(v, x, [1, 1], [1, 1], grid=[40, 2], capacity=16)
    same(a, b)
    assert a["diag"] == b["diag"]  # nothing was loaded for a cell that is left at its first gather
    r = W.rng(62)
    t, d = r.random(n // 2) * 2 * np.pi, 0.01 * np.sqrt(r.random(n // 2))
    x[: n // 2] = np.stack([0.4 + d * np.cos(t), 0.6 + d * np.sin(t)], 1)
    for per in ([1, 1], [0, 0]):
        a, b = run(v, x, [1, 1], per), run(v, x, [1, 1], per, capacity=16)
        same(a, b)
        assert 1.0 < a["diag"]["cuts"] / b["diag"]["cuts"]


@pytest.mark.parametrize("opt", [dict(chunk=1), dict(chunk=4), dict(chunk=64), dict(chunk=65), dict(chunk=2**31 - 1),
                                 dict(waves=5), dict(waves=5, chunk=100)])
def test_chunk_and_waves_by_lane(v, opt):
    """Grabs and waves set by hand never change a cell."""
    n = 80_001
    x = W.uniform(n, 2, 1.0, 71)
    ref, got = run(v, x, [1, 1], [1, 1]), run(v, x, [1, 1], [1, 1], **opt)
    for k in ref:
        if k != "diag":
            assert np.array_equal(got[k], ref[k]), k
    assert got["diag"] == ref["diag"]
