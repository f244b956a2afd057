"""The 2D kernel with one cell per lane, which takes sets of 80,000 particles
and more: against the kernel with eight lanes per cell (a vertex capacity, here
that kernel's own, selects it) on every cell, and against the oracle on some.
Volumes and centroids to 1e-12 of the cell, as every form is held to."""
import numpy as np
import pytest

import oracle
from paper_2209_11606_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

N = 80_000


@pytest.fixture(scope="module")
def v():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_11606_amd import vorohip
    return vorohip


def run(v, x, per, radii=None, **opt):
    xt = torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")
    return v.tessellate(xt, [0, 0], [1, 1], per, v.VC_ALL | v.VC_PERIMETER, radii=radii, **opt)


def same(a, b, live):
    for k in ("nv", "ne", "nf", "nbr_off", "nbr_ids", "nbr_sh"):
        assert np.array_equal(a[k], b[k]), k
    assert np.max(np.abs(a["vol"] - b["vol"])[live] / b["vol"][live]) <= 1e-12
    assert np.max(np.abs(a["cen"] - b["cen"])[live].max(1) / np.sqrt(b["vol"][live])) <= 1e-12
    assert np.max(np.abs(a["perim"] - b["perim"])[live] / b["perim"][live]) <= 1e-12


# the default grid, coarse grids (several periods, dense blocks), a clip square
@pytest.mark.parametrize("n,per,opt", [(N, [1, 1], {}), (N + 1, [0, 0], {}), (N + 63, [1, 0], {}),
                                       (N, [1, 1], dict(grid=[40, 2])), (N, [0, 1], dict(clip=0.004))])
def test_lane_kernel(v, n, per, opt):
    x = W.uniform(n, 2, 1.0, 700 + n)
    a = run(v, x, per, **opt)
    same(a, run(v, x, per, capacity=16, **opt), np.ones(n, bool))
    f = run(v, x, per, precision=v.VC_F32_FILTER, **opt)
    for k in ("vol", "cen", "perim", "nf", "status", "nbr_ids", "nbr_sh"):
        assert np.array_equal(a[k], f[k]), k
    idx = np.arange(0, n, 997)
    r = oracle.Oracle(x, [0, 0], [1, 1], per, **opt).cells(idx, nthreads=oracle.num_threads())
    assert np.array_equal(a["nf"][idx], r["nf"])
    assert np.max(np.abs(a["vol"][idx] - r["vol"]) / r["vol"]) <= 1e-12


def test_lane_kernel_radical(v):
    """Radii up to the mean spacing: some cells are empty or miss their particle.
    Equal radii give the plain cells bit for bit."""
    x = W.uniform(N, 2, 1.0, 811)
    rad = W.rng(812).random(N) * N ** -0.5
    a, b = run(v, x, [1, 1], rad), run(v, x, [1, 1], rad, capacity=16)
    assert np.array_equal(a["status"] == v.VC_CELL_EMPTY, b["status"] == v.VC_CELL_EMPTY)
    assert np.any(a["status"] == v.VC_CELL_EMPTY)
    for k in ("nf", "nbr_off", "nbr_ids", "nbr_sh"):
        assert np.array_equal(a[k], b[k]), k
    # slivers: an absolute floor beside the relative bound, as for every form
    assert np.max(np.abs(a["vol"] - b["vol"]) / (b["vol"] * 1e-12 + 1e-14 / N)) <= 1.0
    plain, equal = run(v, x, [1, 1]), run(v, x, [1, 1], np.full(N, 0.01))
    for k in ("vol", "cen", "perim", "nbr_ids"):
        assert np.array_equal(plain[k], equal[k]), k


def test_lane_kernel_exact_and_subset(v):
    """A lattice (every cell with four-line vertices), and a subset with every
    decision forced through the exact predicate: the cells of the whole set."""
    m = 284
    g0 = np.stack(np.meshgrid(np.arange(m), np.arange(m), indexing="ij"), -1).reshape(-1, 2)
    out = run(v, (g0 + 0.5) / 512.0, [0, 0], clip=1.0 / 512.0)
    assert np.all(out["vol"] == 1.0 / 512.0 ** 2) and set(out["nf"]) == {4}
    x = W.uniform(N, 2, 1.0, 813)
    base = run(v, x, [1, 1])
    ids = np.arange(5, N, 401)
    xt = torch.from_numpy(x).to("cuda:0")
    for force in (0, v.VC_FORCE_EXACT):
        c = v.vc_container_create(xt, v.vc_options_init(2, [0, 0], [1, 1], [1, 1], force=force))
        r = v.vc_result_create(c, v.VC_ALL | v.VC_PERIMETER)
        try:
            v.vc_compute_subset(c, r, ids)
            got = v.fetch(r, v.VC_ALL | v.VC_PERIMETER, N, 2)
        finally:
            v.vc_result_destroy(r)
            v.vc_container_destroy(c)
        for k in ("vol", "cen", "perim", "nv", "nf", "status"):
            assert np.array_equal(got[k][ids], base[k][ids]), (force, k)


def test_lane_kernel_radical_duplicates(v):
    """Coincident particles in a radical set, some of them with an empty cell:
    duplicate or empty as the eight-lane kernel says, particle by particle."""
    x = W.uniform(N, 2, 1.0, 821)
    rad = W.rng(822).random(N) * N ** -0.5
    idx = W.rng(823).permutation(N)
    x[idx[:20_000]] = x[idx[20_000:40_000]]
    a, b = run(v, x, [1, 1], rad), run(v, x, [1, 1], rad, capacity=16)
    kinds = [v.VC_CELL_OK, v.VC_CELL_DUPLICATE, v.VC_CELL_EMPTY]
    assert all(np.any(b["status"] == k) for k in kinds)
    for k in kinds[1:]:
        assert np.array_equal(a["status"] == k, b["status"] == k), k
    for k in ("nf", "nbr_off", "nbr_ids", "nbr_sh"):
        assert np.array_equal(a[k], b[k]), k
