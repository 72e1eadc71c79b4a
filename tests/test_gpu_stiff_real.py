"""GPU: the real solve on a grid with a penalty on one edge (see test_gpu_stiff.py): the sequence takes
its direction up, ends in about the steps of CG with the direction (the oracle's; a quarter and
ten more) and x_0 meets the tolerance by its true residual, verified or not.

In single precision the direction is carried from the start; x_0 then misses the true residual
by what the matrix's own rounding to single precision leaves, eps |A| |x|, so the penalties stay
below that: 6e-8 times the penalty's row, |x| = 1 / penalty there, is 6e-8 of b.
"""
import numpy as np
import pytest

import oracle as O
from test_gpu_stiff import grid

pytestmark = pytest.mark.gpu


def _solve(csr, sigma, cuda, **kw):
    from paper_1102_2143_amd import Operator
    b = np.random.default_rng(721).standard_normal(csr[3])
    op = Operator(*csr, kind="herm", device=cuda)
    op.set_shifts(sigma)
    x, info = op.solve_real(b, check=False, **kw)
    x = x.cpu().numpy()
    op.close()
    rel = [np.linalg.norm(b - O.shifted_apply("herm", *csr)(x[k].astype(complex), s)) / np.linalg.norm(b)
           for k, s in enumerate(sigma)]
    ref = O.cg_m(O.shifted_apply("herm", *csr), b.astype(complex), np.array(sigma), tol=kw["tol"])
    print(f"[gpu] {kw} iters={info['iters']} oracle={ref['iters']} {info['status']} "
          + " ".join(f"{r:.1e}" for r in rel), flush=True)
    return info, rel, ref


@pytest.mark.parametrize("steps", [1, 8])
@pytest.mark.parametrize("verify", [True, False])
@pytest.mark.parametrize("sigma", [[0.0], [1.0, 0.0, 0.0]])
@pytest.mark.parametrize("penalty", [0.0, 1e6, 1e8, 1e10, 1e12, 1e14])
def test_fp64(cuda, penalty, sigma, verify, steps):
    info, rel, ref = _solve(grid(60, 1e-3, penalty), sigma, cuda, tol=1e-10, verify=verify,
                            update_steps=steps)
    assert info["iters"] <= 1.25 * ref["iters"] + 10
    assert rel[sigma.index(0.0)] <= 1.05e-10
    # the other shifts' residuals are implied, and the stiff rows' rounding is in them
    if not verify or max(rel) <= 1e-10:
        assert info["status"] == "ok"
    else:
        assert info["status"] in ("ok", "notconv")


@pytest.mark.parametrize("verify", [True, False])
@pytest.mark.parametrize("penalty", [0.0, 1e2, 1e4])
def test_single(cuda, penalty, verify):
    info, rel, ref = _solve(grid(60, 1e-3, penalty), [0.0], cuda, tol=1e-5, prec="mixed", verify=verify)
    assert info["status"] == "ok" and info["iters"] <= 1.25 * ref["iters"] + 10
    assert rel[0] <= 1.05e-5


@pytest.mark.parametrize("prec,tol", [("fp64", 1e-10), ("mixed", 1e-5)])
@pytest.mark.parametrize("penalty", [0.0, 1e8])
def test_not_positive_definite(cuda, penalty, prec, tol):
    info, _, _ = _solve(grid(20, 1e-3, penalty), [-0.5, 0.1], cuda, tol=tol, prec=prec)
    assert info["status"] == "breakdown"
