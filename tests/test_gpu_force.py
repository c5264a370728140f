"""Link force in the row layout: infinities stay what they are on the planes, and a step on
few columns takes no longer than there."""
import numpy as np
import pytest

from paper_1710_09745_amd import synth

from gpu_util import best_times, context, inputs, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [5, 8, 11, 16, 20, 33])
def test_row_force_keeps_infinities(n):
    """An infinite number in the last column: its lane's neighbours past that column, which
    hold a copy of it, add nothing (0 x infinity would turn the sums into NaN)."""
    dims = (6, 6, 6, 10)
    fat, lng, X = inputs(dims, True, n, 25000 + n)
    Lam = synth.rhs(synth.make_rng(25100 + n), n, dims)
    X[n - 1, 100, 1] = np.inf + 1j
    out = []
    for planes in (0, 1):
        ctx = context(dims, True, fat, lng, 0.1)
        ctx.set_option("site_order", planes)
        out.append([g.cpu().numpy() for g in ctx.link_force(to_dev(X), to_dev(Lam))])
        ctx.close()
    for rows, planes in zip(*out):
        for a, b in ((rows.real, planes.real), (rows.imag, planes.imag)):
            assert np.array_equal(np.isnan(a), np.isnan(b)) and np.array_equal(np.isinf(a), np.isinf(b))
            assert np.isinf(a).any()
            ok = np.isfinite(b)
            assert np.abs(a[ok] - b[ok]).max() <= 1e-12 * np.abs(b[ok]).max()


def test_row_force_on_five_columns_takes_no_longer_than_planes():
    """16^4: 1.22 times as long with the streaming hint on half rows; the margin is for the
    clock."""
    dims, n = (16, 16, 16, 16), 5
    fat, lng, X = inputs(dims, True, n, 25200)
    x = to_dev(X)
    rows, planes = (context(dims, True, fat, lng, 0.05) for _ in range(2))
    planes.set_option("site_order", 1)
    t = best_times({"rows": lambda: rows.link_force(x, x), "planes": lambda: planes.link_force(x, x)}, repeats=50)
    assert t["rows"] <= 1.13 * t["planes"]
