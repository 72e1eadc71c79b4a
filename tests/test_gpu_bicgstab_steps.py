"""GPU: the two-kernel BiCGStab-M iteration at its edges, against the oracle.

Steps of the shifts are composed four at a time: stops before, at and after an
application, on the sliced copy (16- and 32-bit columns) and on the CSR, grids that fill
whole slices and that leave a partial one, 64 shifts.

Tolerances: after at most ten steps both take the same steps up to rounding; the parity
test after five steps holds 1e-12, and each five further ones are granted a decade.
Converged solutions: 1e-8, as the other parity tests.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def _problem(dims, ns):
    rowptr, col, vals = W.laplacian7_csr(dims, 79)
    n = int(np.prod(dims))
    # unequal couplings towards the two neighbours of a row: not Hermitian
    upper = col > np.repeat(np.arange(n), np.diff(rowptr))
    vals = vals + 0.3 * upper * (vals == -1.0) + 0.05j * upper
    return dict(csr=(rowptr, col, vals, n), b=W.gaussian_rhs(n, 80),
                sigma=W.logspace_shifts(1e-2, 2.0, ns),
                apply=O.shifted_apply("general", rowptr, col, vals, n))


def _solve(p, cuda, **kw):
    from paper_1102_2143_amd import Operator
    op = Operator(*p["csr"], kind="general", device=cuda)
    op.set_shifts(p["sigma"])
    x, info = op.solve_bicgstab(p["b"], **kw)
    x = x.cpu().numpy()
    op.close()
    return x, info


def _rel(a, b):
    return (np.linalg.norm(a - b, axis=-1) / np.linalg.norm(b, axis=-1)).max()


@pytest.mark.parametrize("fmt", ["sell", "sell32", "csr"])
@pytest.mark.parametrize("limit", [1, 3, 4, 5, 8, 9])
def test_stops_around_an_application(cuda, limit, fmt):
    p = _problem((7, 6, 5), 5)
    x, info = _solve(p, cuda, tol=1e-30, max_iter=limit, poll_every=3, format=fmt)
    ref = O.bicgstab_m(p["apply"], p["b"], p["sigma"], tol=0.0, max_iter=limit)
    assert info["status"] == "notconv" and info["iters"] == limit
    assert _rel(x, ref["x"]) <= 1e-11


@pytest.mark.parametrize("fmt", ["auto", "csr"])
@pytest.mark.parametrize("dims,ns", [((8, 8, 4), 3), ((5, 13, 5), 64), ((17, 16, 15), 7)])
def test_converged(cuda, dims, ns, fmt):
    p = _problem(dims, ns)
    x, info = _solve(p, cuda, tol=1e-11, format=fmt)
    ref = O.bicgstab_m(p["apply"], p["b"], p["sigma"], tol=1e-11)
    assert info["status"] == "ok" and abs(info["iters"] - ref["iters"]) <= 2
    assert np.all(np.abs(info["freeze_iter"] - ref["freeze_iter"]) <= 2)
    assert _rel(x, ref["x"]) <= 1e-8


def test_no_steps(cuda):
    p = _problem((5, 4, 3), 4)
    x, info = _solve(p, cuda, max_iter=0)
    assert info["iters"] == 0 and not x.any()
