"""GPU parity of the row-layout kernels (more than 4 right-hand sides) at the edges of
their tiles: half rows (5 to 8 columns), one to four 16-column tiles with and without a
remainder, site counts that leave ragged 16- and 32-site blocks, extents of 2 and 4
(neighbours that wrap twice), and lattices that take the per-XCD cell walk."""
import numpy as np
import pytest

import oracle

from gpu_util import col_rel_err, context, elem_rel_err, inputs, to_dev

pytestmark = pytest.mark.gpu

LATTICES = [((2, 2, 2, 4), True), ((6, 6, 2, 6), False), ((6, 6, 6, 2), True), ((8, 8, 8, 4), True)]


@pytest.mark.parametrize("n", [5, 8, 9, 16, 17, 32, 48, 64])
@pytest.mark.parametrize("dims,improved", LATTICES)
def test_row_apply_matches_oracle(dims, improved, n):
    fat, lng, B = inputs(dims, improved, n, 11000 + n)
    ctx = context(dims, improved, fat, lng, 0.07)
    ref = oracle.Operator(dims, fat, lng, 0.07).apply(B)
    got = ctx.apply(to_dev(B)).cpu().numpy()
    # the tolerance of every FP64 operator test: 16 terms of three complex products in
    # another order
    assert col_rel_err(got, ref).max() <= 1e-12
    assert elem_rel_err(got, ref).max() <= 1e-12


@pytest.mark.parametrize("n", [2, 5])
def test_reloaded_links_reach_both_layouts(n):
    """New links replace those of both layouts: the plane copy (up to 4 columns) is made
    from the row copy on first use and again after a reload."""
    dims = (4, 4, 4, 6)
    ctx = None
    for seed in (11500, 11600):
        fat, lng, B = inputs(dims, True, n, seed)
        if ctx is None:
            ctx = context(dims, True, fat, lng, 0.07)
        else:
            ctx.load_links(fat, lng)
        ref = oracle.Operator(dims, fat, lng, 0.07).apply(B)
        assert elem_rel_err(ctx.apply(to_dev(B)).cpu().numpy(), ref).max() <= 1e-12
