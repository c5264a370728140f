"""Rounding of the operator in the row layout, against its definition in extended precision:
no larger than in the lane-split kernel of the plane layout, which sums four chains."""
import numpy as np
import pytest

import oracle

from gpu_util import best_times, context, emulated_sloppy_apply, inputs, site_scaled_err, to_dev
from test_gpu_operator import SLOPPY_TOL

pytestmark = pytest.mark.gpu


def _apply_extended(dims, fat, lng, mass, B):
    """A B = 4 m^2 B - D_eo D_oe B with numpy's long double (64 bits of mantissa)."""
    shape = dims[::-1]  # site index: x fastest
    t, z, y, x = np.indices(shape)
    odd = (x + y + z + t) % 2 == 1
    # eta_x = 1, eta_y = (-1)^x, eta_z = (-1)^(x+y), eta_t = (-1)^(x+y+z)
    eta = [1 - 2 * (s % 2) for s in (0 * x, x, x + y, x + y + z)]

    def D(psi):  # [*shape, 3, N]
        out = np.zeros_like(psi)
        for d, U in ((1, fat), (3, lng)):
            for mu in range(4):
                ax = 3 - mu
                u = U[mu].reshape(*shape, 3, 3).astype(np.clongdouble)
                e = eta[mu][..., None, None]
                back = np.roll(u, d, axis=ax).conj().swapaxes(-1, -2)
                for w, s in ((e * u, np.roll(psi, -d, axis=ax)), (-e * back, np.roll(psi, d, axis=ax))):
                    for b in range(3):
                        out += w[..., :, b, None] * s[..., None, b, :]
        return out

    n = B.shape[0]
    full = np.zeros((*shape, 3, n), dtype=np.clongdouble)
    full[~odd] = B.transpose(1, 2, 0)
    ddd = D(np.where(odd[..., None, None], D(full), 0))
    return (4 * np.longdouble(mass) ** 2 * full - ddd)[~odd].transpose(2, 0, 1)


def test_row_operator_rounds_no_more_than_the_planes():
    dims, n = (8, 8, 8, 8), 17  # a full and a partial tile of columns
    fat, lng, B = inputs(dims, True, n, 23000)
    ref = _apply_extended(dims, fat, lng, 0.05, B)
    err = {}
    for planes in (0, 1):
        ctx = context(dims, True, fat, lng, 0.05)
        ctx.set_option("hop_kernel", planes)
        for m in (5, n):
            x = to_dev(B[:m])
            for prec, got in (("fp64", ctx.apply(x)), ("fp32", ctx.apply_prec("fp32", x))):
                d = got.cpu().numpy() - ref[:m]
                err[planes, m, prec] = float(np.sqrt((np.abs(d) ** 2).sum() / (np.abs(ref[:m]) ** 2).sum()))
        ctx.close()
    print(err)
    for m in (5, n):
        for prec in ("fp64", "fp32"):
            # root mean squares over 30720 numbers and more: within 1 % of their expectation
            assert err[0, m, prec] <= 1.02 * err[1, m, prec]


@pytest.mark.parametrize("prec", ["fp32", "fix16", "bf16"])
@pytest.mark.parametrize("dims,n", [((6, 6, 6, 10), 5), ((6, 6, 6, 10), 20), ((16, 16, 16, 20), 6),
                                    ((16, 16, 16, 20), 7)])
def test_sloppy_apply_on_either_side_of_its_layout_rule(prec, dims, n):
    """Rows and planes (16-bit formats on 5 and 6 columns above 32768 sites of a parity)
    against the oracle's emulation of the storage."""
    fat, lng, B = inputs(dims, True, n, 23100 + n)
    ctx = context(dims, True, fat, lng, 0.05)
    ref = emulated_sloppy_apply(oracle.Operator(dims, fat, lng, 0.05), prec, B)
    # the storage roundings of the operator's tests
    assert site_scaled_err(ctx.apply_prec(prec, to_dev(B)).cpu().numpy(), ref) <= SLOPPY_TOL[prec]


def test_sloppy_apply_takes_no_longer_than_planes():
    """16^3 x 48, 5 columns in 16-bit storage: 1.17 times as long in rows; the margin is for
    the clock."""
    dims, n = (16, 16, 16, 48), 5
    fat, lng, B = inputs(dims, True, n, 23200)
    x = to_dev(B)
    default, planes = (context(dims, True, fat, lng, 0.05) for _ in range(2))
    planes.set_option("site_order", 1)
    t = best_times({"default": lambda: default.apply_prec("fix16", x),
                    "planes": lambda: planes.apply_prec("fix16", x)}, repeats=50)
    assert t["default"] <= 1.1 * t["planes"]
