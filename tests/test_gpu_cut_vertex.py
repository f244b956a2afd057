"""Vertices of the grouped kernel, whose reciprocal is no division: against the
one-cell kernel's, which divides, and over the boxes it holds for."""
import numpy as np
import pytest

from paper_2209_11606_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def v():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_11606_amd import vorohip
    return vorohip


def test_volumes_of_both_kernels(v):
    """400 walled sets of 24 particles: with one batch of candidates a cell, both
    kernels make the same cuts in the same lanes, and add the same volume terms in
    the same order, so equal vertices give equal bits (cells of up to 32 vertices)."""
    t, n = 400, 24
    x = torch.from_numpy(W.rng(5).random((t * n, 3))).to("cuda:0")
    out = []
    for form in (dict(), dict(cells_per_wave=2)):
        opts = [v.vc_options_init(3, [0] * 3, [1] * 3, [0] * 3, grid=[1, 1, 1], **form)] * t
        b = v.vc_batch_create(x, np.arange(0, t * n + 1, n), opts)
        r = v.vc_batch_result_create(b, v.VC_ALL)
        try:
            v.vc_batch_compute(b, r, False)
            out.append(v.fetch(r, v.VC_ALL, t * n, 3))
        finally:
            v.vc_result_destroy(r)
            v.vc_batch_destroy(b)
    a, g = out
    assert np.array_equal(a["nf"], g["nf"]) and np.array_equal(a["nv"], g["nv"])
    k = (a["nv"] <= 32) & (g["status"] == 0)
    assert k.sum() > 9000 and np.array_equal(a["vol"][k], g["vol"][k])


@pytest.mark.parametrize("per", [[0, 0, 0], [1, 1, 1]])
@pytest.mark.parametrize("e", [-240, -100, 100, 240])
def test_scaled_boxes(v, per, e):
    """Scaling by a power of two changes no mantissa while nothing under- or
    overflows: |q|^2 h and volumes lie within 2^-960 .. 2^960 here."""
    x, s = W.uniform(500, 3, 1.0, 9), 2.0 ** e
    a, b = (v.tessellate(torch.from_numpy(x * c).to("cuda:0"), [0] * 3, [c] * 3, per, v.VC_ALL, cells_per_wave=2)
            for c in (1.0, s))
    for k in ("status", "nv", "ne", "nf", "nbr_ids"):
        assert np.array_equal(a[k], b[k]), k
    assert np.array_equal(a["vol"] * s * s * s, b["vol"]) and np.array_equal(a["cen"] * s, b["cen"])
