"""GPU: the real multishift solve's one-kernel iteration at its edges, against the oracle.

Steps of the shifted update are composed and applied together: every number of folded
steps, stops before, at and after an application, 64 shifts, grids of one row, of a
partial slice and of one row more than whole slices, b = 0.  The oracle takes the same
number of steps, so its iterates are the same up to rounding: eps times the steps (20 at
most) times the condition number (below 9 / 0.01) is 4e-12, and 1e-8 where both run to
tol 1e-10 (as the other parity tests).
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def _problem(nx, ny, ns):
    rowptr, col, vals = W.poisson5pt_csr(nx, ny)
    n = nx * ny
    return dict(csr=(rowptr, col, vals, n), b=np.random.default_rng(78).standard_normal(n),
                sigma=W.logspace_shifts(1e-2, 1.0, ns),
                apply=O.shifted_apply("herm", rowptr, col, vals, n))


def _solve(p, cuda, **kw):
    from paper_1102_2143_amd import Operator
    op = Operator(*p["csr"], kind="herm", device=cuda)
    op.set_shifts(p["sigma"])
    x, info = op.solve_real(p["b"], **kw)
    x = x.cpu().numpy()
    op.close()
    return x, info


def _rel(a, b):
    return (np.linalg.norm(a - b, axis=-1) / np.linalg.norm(b, axis=-1)).max()


@pytest.mark.parametrize("steps", [1, 2, 3, 7, 8])
@pytest.mark.parametrize("limit", [1, 7, 8, 9, 16, 20])
def test_stops_around_an_application(cuda, limit, steps):
    p = _problem(13, 11, 6)
    x, info = _solve(p, cuda, max_iter=limit, update_steps=steps)
    ref = O.cg_m(p["apply"], p["b"].astype(complex), p["sigma"], max_iter=limit)
    assert info["status"] == "notconv" and info["iters"] == limit
    assert _rel(x, ref["x"].real) <= 4e-12


@pytest.mark.parametrize("prec,bar", [("fp64", 1e-8), ("mixed", 2e-4)])
@pytest.mark.parametrize("nx,ny,ns", [(1, 1, 3), (13, 5, 2), (8, 8, 64), (16, 65, 15)])
def test_sizes_and_shifts(cuda, nx, ny, ns, prec, bar):
    # single precision stops at 1e-6; its error is within the condition number of that
    tol = 1e-10 if prec == "fp64" else 1e-6
    p = _problem(nx, ny, ns)
    x, info = _solve(p, cuda, tol=tol, prec=prec, verify=False)
    ref = O.cg_m(p["apply"], p["b"].astype(complex), p["sigma"], tol=tol)
    assert info["status"] == "ok" and abs(info["iters"] - ref["iters"]) <= 2
    exact = O.dense_solve("herm", *p["csr"], p["b"].astype(complex), p["sigma"]).real
    assert _rel(x, exact) <= bar


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_zero_rhs_and_no_steps(cuda, prec):
    p = _problem(13, 5, 4)
    x, info = _solve(p, cuda, max_iter=0, prec=prec)
    assert info["iters"] == 0 and not x.any()
    p["b"] = np.zeros_like(p["b"])
    x, info = _solve(p, cuda, prec=prec)
    assert info["status"] == "ok" and info["iters"] == 0 and not x.any()
