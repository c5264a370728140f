"""Pseudo-block CG: iterates at the edges of its launch rules (block sums of the hop read
directly or folded first, 16 to 128 lanes a column, x with r or with p on planes), and the
row layout against the planes in time where few sites have many columns."""
import numpy as np
import pytest

import oracle
from paper_1710_09745_amd import bcg

from gpu_util import best_times, col_rel_err, context, inputs, to_dev

pytestmark = pytest.mark.gpu


# 4096 sites: dots read directly, update 1 in 48 to 512 workgroups; 10240: dots folded;
# one column and 3 above 8192 sites: planes, 18432 sites: x with p
@pytest.mark.parametrize("dims,n", [((4, 4, 4, 4), 1), ((4, 4, 4, 4), 2), ((8, 8, 8, 16), 4), ((8, 8, 8, 16), 24),
                                    ((8, 8, 8, 16), 64), ((16, 16, 8, 10), 9), ((16, 16, 8, 10), 3),
                                    ((16, 16, 12, 12), 2), ((16, 16, 12, 12), 33)])
def test_pseudo_iterates_match_oracle_cg(dims, n):
    k = 3
    fat, lng, B = inputs(dims, True, n, 24000 + n)
    ctx = context(dims, True, fat, lng, 0.1, tol=1e-14, max_iter=k)
    X, info = ctx.solve_pseudo(to_dev(B), raise_on_error=False)
    assert info["rc"] == bcg.ERR_NOT_CONVERGED and info["iters"] == k
    op = oracle.Operator(dims, fat, lng, 0.1)
    ref = np.stack([oracle.cg(op.apply, B[i], 1e-14, max_iter=k)[0] for i in range(n)])
    # the bound of the row layout's iterates
    assert col_rel_err(X.cpu().numpy(), ref).max() <= 1e-10


@pytest.mark.parametrize("dims,n", [((4, 4, 4, 4), 3), ((8, 8, 8, 8), 20)])
def test_pseudo_columns_finish_one_by_one(dims, n):
    """Every column stops at its own iteration while the others go on."""
    fat, lng, B = inputs(dims, True, n, 24100 + n)
    ctx = context(dims, True, fat, lng, 0.2, tol=1e-9)
    X, info = ctx.solve_pseudo(to_dev(B))
    op = oracle.Operator(dims, fat, lng, 0.2)
    res = B - op.apply(X.cpu().numpy())
    rel = np.linalg.norm(res.reshape(n, -1), axis=1) / np.linalg.norm(B.reshape(n, -1), axis=1)
    assert rel.max() <= 1e-9


@pytest.mark.parametrize("n", [24, 64])
def test_rows_take_no_longer_than_planes_on_a_small_lattice(n):
    """8^4: row kernels whose grid counted sites alone took 1.6 (N = 24) and 2.4 times (N = 64)
    as long as the planes'; the margin is for the clock."""
    dims = (8, 8, 8, 8)
    fat, lng, B = inputs(dims, True, n, 24200)
    x = to_dev(B)
    rows, planes = (context(dims, True, fat, lng, 0.05, tol=1e-14, max_iter=60) for _ in range(2))
    planes.set_option("site_order", 1)
    t = best_times({"rows": lambda: rows.solve_pseudo(x, raise_on_error=False),
                    "planes": lambda: planes.solve_pseudo(x, raise_on_error=False)})
    assert t["rows"] <= 1.3 * t["planes"]
