"""GPU: the largest limits that fit their fields mean "no limit": the host's own bounds on what it
queues are above them, so every solve runs to its tolerance."""
import numpy as np
import pytest
import torch

import workloads as W

pytestmark = pytest.mark.gpu

NO_LIMIT = 2**31 - 1


def _kw(verify, **kw):
    return dict(max_iter=NO_LIMIT, refine_max_iter=NO_LIMIT, verify=verify, **kw)


def _check(op, x, b, info, tol):
    assert info["status"] == "ok" and info["iters"] > 0
    for k, s in enumerate(op.sigma):
        r = op.apply(x[k], float(s)).cpu().numpy() - b
        assert np.linalg.norm(r) <= 2 * tol * np.linalg.norm(b)


@pytest.mark.parametrize("verify", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_solve_and_batch(cuda, prec, verify):
    from paper_1102_2143_amd import Operator
    from paper_1102_2143_amd.api import solve_batched
    op = Operator.staggered(W.random_su3_links((4, 4, 4, 5), 651), (4, 4, 4, 5), 0.1, device=cuda)
    op.set_shifts([0.01, 0.1])
    b = W.gaussian_rhs(op.n, 652)
    x, info = op.solve(b, tol=1e-8, prec=prec, **_kw(verify))
    _check(op, x, b, info, 1e-8)
    xs, infos, status = solve_batched([op], [b[None]], tol=1e-8, prec=prec, **_kw(verify))
    assert status == "ok"
    _check(op, xs[0][0], b, infos[0], 1e-8)
    # the refinement's own limit: a sequence that ends early leaves all of the work to it
    if verify:
        x, info = op.solve(b, tol=1e-8, prec=prec, refine_max_iter=NO_LIMIT, max_iter=3)
        assert info["refine_iters"] > 3
        _check(op, x, b, info, 1e-8)
    op.close()


@pytest.mark.parametrize("verify", [True, False])
def test_real_and_bicgstab(cuda, verify):
    from paper_1102_2143_amd import Operator
    op = Operator(*W.poisson5pt_csr(13, 11), 143, kind="herm", device=cuda)
    op.set_shifts([0.01, 0.1])
    b = np.random.default_rng(653).standard_normal(op.n)
    x, info = op.solve_real(b, tol=1e-8, **_kw(verify))
    _check(op, x.to(dtype=torch.complex128), b, info, 1e-8)
    x, info = op.solve_bicgstab(b, tol=1e-8, **_kw(verify))
    _check(op, x, b, info, 1e-8)
    op.close()
