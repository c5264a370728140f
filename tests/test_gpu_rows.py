"""GPU parity of the row-layout kernels (more than 4 right-hand sides) at the edges of
their tiles: half rows (5 to 8 columns), one to four 16-column tiles with and without a
remainder, site counts that leave ragged 16- and 32-site blocks, extents of 2 and 4
(neighbours that wrap twice), and lattices that take the per-XCD cell walk."""
import numpy as np
import pytest

import oracle
from paper_1710_09745_amd import bcg, synth

from gpu_util import (col_rel_err, context, elem_rel_err, emulated_sloppy_apply, inputs, site_scaled_err, to_dev,
                      true_rel_res)
from test_gpu_operator import SLOPPY_TOL

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


@pytest.mark.parametrize("dims,n", [((16, 16, 16, 24), 20), ((24, 24, 4, 8), 9)])
def test_row_apply_on_larger_lattices(dims, n):
    """Links past the caches (streamed), a second tile of 4 columns, and planes of more than
    256 sites (cells of 4 rows)."""
    fat, lng, B = inputs(dims, True, n, 11300 + n)
    ctx = context(dims, True, fat, lng, 0.07)
    op = oracle.Operator(dims, fat, lng, 0.07)
    assert elem_rel_err(ctx.apply(to_dev(B)).cpu().numpy(), op.apply(B)).max() <= 1e-12
    got = ctx.apply_prec("fp32", to_dev(B)).cpu().numpy()
    assert site_scaled_err(got, emulated_sloppy_apply(op, "fp32", B)) <= SLOPPY_TOL["fp32"]


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


@pytest.mark.parametrize("prec", ["fp32", "fp16", "bf16", "fix16"])
@pytest.mark.parametrize("n", [7, 16, 40])
def test_row_sloppy_apply_matches_emulation(prec, n):
    dims = (6, 6, 4, 6)
    fat, lng, B = inputs(dims, True, n, 12000 + n)
    ctx = context(dims, True, fat, lng, 0.05)
    ref = emulated_sloppy_apply(oracle.Operator(dims, fat, lng, 0.05), prec, B)
    # the storage roundings of the plane kernels' test
    assert site_scaled_err(ctx.apply_prec(prec, to_dev(B)).cpu().numpy(), ref) <= SLOPPY_TOL[prec]


@pytest.mark.parametrize("n", [5, 8, 9, 16, 17, 24, 32, 40, 64])
def test_row_iterates_match_oracle(n):
    """Three iterations with a reliable update forced in (Gram, passes A and B, block
    multiply and column norms at every tile count), FP64 storage and CholQR2."""
    dims = (6, 6, 6, 10)  # 1080 sites: ragged 16- and 32-site blocks
    fat, lng, B = inputs(dims, True, n, 13000 + n)
    ctx = context(dims, True, fat, lng, 0.1, tol=1e-14, ru_delta=0.9, max_iter=3)
    ctx.set_stability(qr_passes=2)
    X, info = ctx.solve(to_dev(B), raise_on_error=False)
    assert info["rc"] == bcg.ERR_NOT_CONVERGED and info["iters"] == 3
    ref, _ = oracle.block_cg_rq(oracle.Operator(dims, fat, lng, 0.1).apply, B, 1e-14, max_iter=3)
    assert col_rel_err(X.cpu().numpy(), ref).max() <= 1e-10


@pytest.mark.parametrize("n", [8, 9])
def test_row_iterates_match_planes_on_a_large_lattice(n):
    """The Gram partials of several rounds of workgroups (above 1024 they are summed in two
    steps): two iterations against the plane kernels."""
    dims = (32, 32, 32, 24 if n > 8 else 48)
    fat, lng, B = inputs(dims, False, n, 13500 + n)
    X = []
    for planes in (0, 1):
        ctx = context(dims, False, fat, lng, 0.3, tol=1e-14, max_iter=2)
        ctx.set_option("site_order", planes)
        x, info = ctx.solve(to_dev(B), raise_on_error=False)
        assert info["iters"] == 2
        X.append(x.cpu().numpy())
    # two well conditioned iterations: the bound of the small lattices' test
    assert col_rel_err(X[0], X[1]).max() <= 1e-10


@pytest.mark.parametrize("prec", ["fp32", "fix16"])
@pytest.mark.parametrize("n", [6, 20, 50])
def test_row_mixed_solve_meets_tolerance(prec, n):
    dims = (8, 8, 8, 6)
    fat, lng, B = inputs(dims, True, n, 14000 + n)
    ctx = context(dims, True, fat, lng, 0.15, tol=1e-9, prec=prec)
    X, _ = ctx.solve(to_dev(B))
    op = oracle.Operator(dims, fat, lng, 0.15)
    assert true_rel_res(op, B, X.cpu().numpy()).max() <= 1e-9


@pytest.mark.parametrize("n", [5, 8, 13, 16, 40, 64])
@pytest.mark.parametrize("dims,improved", LATTICES)
def test_row_link_force_matches_oracle(dims, improved, n):
    fat, lng, X = inputs(dims, improved, n, 15000 + n)
    Lam = synth.rhs(synth.make_rng(15100 + n), n, dims)
    ctx = context(dims, improved, fat, lng, 0.1)
    gf, gl = ctx.link_force(to_dev(X), to_dev(Lam))
    rf, rl = oracle.Operator(dims, fat, lng, 0.1).link_force(X, Lam)
    assert np.abs(gf.cpu().numpy() - rf).max() <= 1e-12 * np.abs(rf).max()
    if improved:
        assert np.abs(gl.cpu().numpy() - rl).max() <= 1e-12 * np.abs(rl).max()


@pytest.mark.parametrize("n", [5, 24, 40])
def test_row_pseudo_block_iterates_match_oracle_cg(n):
    dims, k = (6, 6, 6, 2), 3
    fat, lng, B = inputs(dims, True, n, 16000 + n)
    ctx = context(dims, True, fat, lng, 0.1, tol=1e-14, max_iter=k)
    X, info = ctx.solve_pseudo(to_dev(B), raise_on_error=False)
    assert info["iters"] == k
    op = oracle.Operator(dims, fat, lng, 0.1)
    ref = np.stack([oracle.cg(op.apply, B[i], 1e-14, max_iter=k)[0] for i in range(n)])
    assert col_rel_err(X.cpu().numpy(), ref).max() <= 1e-10
