"""GPU: BiCGStab-M where a stabilising step leaves 1e-9 of the half-step residual.

A is made of blocks [[2, d], [1, 3]] and b lives on each block's first row, so the first
half-step residual is (0, -b/2) and the step with om = 1/3 leaves d/6 of b.  |r|^2 and w^H r by
difference are rounding there; taken from r itself they say that d/6 is above tol, and the
second step ends at rounding (the minimal polynomial has degree two).
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


def _blocks(count, d):
    n = 2 * count
    rowptr = np.arange(0, 2 * n + 1, 2, dtype=np.int64)
    col = np.repeat(np.arange(0, n, 2), 4).reshape(-1, 4) + np.array([0, 1, 0, 1])
    vals = np.tile(np.array([2.0, d, 1.0, 3.0], dtype=complex), count)
    b = np.zeros(n, dtype=complex)
    b[::2] = W.gaussian_rhs(count, 661)
    return (rowptr, col.reshape(-1).astype(np.int32), vals, n), b


@pytest.mark.parametrize("verify", [True, False])
@pytest.mark.parametrize("fmt", ["auto", "csr"])
@pytest.mark.parametrize("d,steps", [(1e-9, 2), (1e-7, 2), (1e-13, 1)])
def test_small_remainder(cuda, d, steps, fmt, verify):
    from paper_1102_2143_amd import Operator
    csr, b = _blocks(400, d)
    op = Operator(*csr, kind="general", device=cuda)
    op.set_shifts([0.0, 0.5, 2.0])
    x, info = op.solve_bicgstab(b, tol=1e-11, format=fmt, verify=verify)
    assert info["status"] == "ok" and info["iters"] == steps, info
    x = x.cpu().numpy()
    for k, s in enumerate((0.0, 0.5, 2.0)):
        inv = np.linalg.inv(np.array([[2.0 + s, d], [1.0, 3.0 + s]]))
        exact = (b.reshape(-1, 2) @ inv.T).reshape(-1)
        assert np.linalg.norm(x[k] - exact) <= 1e-10 * np.linalg.norm(exact)
    op.close()
