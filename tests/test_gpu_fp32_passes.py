"""FP32 storage on 17 to 32 columns: the passes of an iteration form their sums in FP64 and
round once, as a result is stored.  The operator here is exact in FP32 but for one rounding
of each hop (one direction of unit links, 4 m^2 = 1), so the oracle's formulas with the same
roundings give the same stored numbers; only the arithmetic of the passes is left to differ."""
import numpy as np
import pytest

import oracle
from paper_1710_09745_amd import bcg, synth

from gpu_util import col_rel_err, context, to_dev

pytestmark = pytest.mark.gpu

DIMS = (10, 6, 6, 6)  # three distinct eigenvalues between 1 and 5; ragged 16-site blocks


def _fl(M):
    return M.astype(np.complex64).astype(np.complex128)


def _gram(A, B):
    """A^H B as the kernels keep it: tiles of 16 above the diagonal, their conjugates below,
    the Hermitian part of the diagonal tiles."""
    G = A.conj().T @ B
    n = G.shape[0]
    out = np.empty_like(G)
    for a in range(0, n, 16):
        for b in range(0, n, 16):
            g, h = G[a:a + 16, b:b + 16], G[b:b + 16, a:a + 16].conj().T
            out[a:a + 16, b:b + 16] = g if a < b else (h if a > b else 0.5 * (g + h))
    return out


def _emulated(op, B, iters):
    vh = B.shape[1]
    hop = lambda p, M: oracle.to_mat(op.hop(p, oracle.from_mat(M, vh)))
    R = oracle.to_mat(B)
    C = oracle.cholesky_upper(_gram(R, R))
    Q = P = _fl(R @ np.linalg.inv(C))
    X = np.zeros_like(R)
    for _ in range(iters):
        T = _fl(hop(1, P))
        AP = _fl(P - _fl(hop(0, T)))
        beta = np.linalg.inv(_gram(P, AP))
        X = X + P @ (beta @ C)
        Q = _fl(Q - AP @ beta)
        S = oracle.cholesky_upper(_gram(Q, Q))
        C = S @ C
        Q = _fl(Q @ np.linalg.inv(S))
        P = _fl(Q + P @ S.conj().T)
    return oracle.from_mat(X, vh)


@pytest.mark.parametrize("n", [17, 24, 25, 32])
def test_fp32_passes_sum_in_fp64(n):
    V = int(np.prod(DIMS))
    fat = np.zeros((4, V, 3, 3), dtype=np.complex128)
    fat[0] = np.eye(3)
    B = synth.rhs(synth.make_rng(22000 + n), n, DIMS)
    ctx = context(DIMS, False, fat, None, 0.5, tol=1e-14, prec="fp32", ru_delta=0.0, max_iter=2)
    X, info = ctx.solve(to_dev(B), raise_on_error=False)
    assert info["rc"] == bcg.ERR_NOT_CONVERGED and info["iters"] == 2
    ref = _emulated(oracle.Operator(DIMS, fat, None, 0.5), B, 2)
    # FP64 rounding differences (1e-13 of a number) move about one stored number in a
    # million by one FP32 unit: below 1e-10, times the condition number of 5; sums in FP32
    # give 1e-8 and more
    assert col_rel_err(X.cpu().numpy(), ref).max() <= 2e-9
