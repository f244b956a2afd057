"""Cells per queue grab and the number of waves follow the number of cells
when they are left to the library: around the sizes where the rule changes,
every form gives the same bits as with both set by hand."""
import numpy as np
import pytest

from paper_2209_11606_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FORMS = [dict(dim=3), dict(dim=3, cells_per_wave=2), dict(dim=3, cells_per_wave=4), dict(dim=2)]


@pytest.fixture(scope="module")
def v():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2209_11606_amd import vorohip
    return vorohip


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n", [1, 3, 127, 1025, 40961])
def test_rule_keeps_cells(v, form, n):
    form = dict(form)
    dim = form.pop("dim")
    x = torch.from_numpy(W.uniform(n, dim, 1.0, 500 + n)).to("cuda:0")
    box = ([0] * dim, [1] * dim, [1] * dim)
    mask = v.VC_VOLUME | v.VC_CENTROID | v.VC_COUNTS | v.VC_NEIGHBORS
    ref = v.tessellate(x, *box, mask, waves=33, chunk=7, **form)
    for opt in (dict(), dict(waves=2), dict(chunk=1)):
        got = v.tessellate(x, *box, mask, **form, **opt)
        for k in ref:
            if k != "diag":
                assert np.array_equal(got[k], ref[k]), (k, opt)
