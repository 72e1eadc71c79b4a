"""GPU: a right-hand side whose |b|^2 is not finite is a breakdown, with x = 0, on every path of
the solves: an infinite or NaN entry, and finite entries whose squares overflow."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

RHS = {"inf": lambda b: np.where(np.arange(b.size) == 5, np.inf, b),
       "nan": lambda b: np.where(np.arange(b.size) == 5, np.nan, b),
       "large": lambda b: 1e160 * b}


def _links(dims, cuda):
    from paper_1102_2143_amd import Operator
    return Operator.staggered(W.random_su3_links(dims, 641), dims, 0.1, device=cuda)


def _grid(cuda):
    from paper_1102_2143_amd import Operator
    return Operator(*W.poisson5pt_csr(13, 11), 143, kind="herm", device=cuda)


PATHS = {"one workgroup": (lambda c: _links((4, 4, 4, 4), c), {}),
         "links": (lambda c: _links((4, 4, 4, 5), c), {}),
         "sliced": (lambda c: _links((4, 4, 4, 5), c), dict(format="sell")),
         "csr": (lambda c: _links((4, 4, 4, 5), c), dict(format="csr")),
         "sliced, A given": (_grid, {}),
         "csr, A given": (_grid, dict(format="csr"))}


def _broke_down(x, info):
    assert info["status"] == "breakdown" and info["iters"] == 0, info
    assert not bool(x.abs().any())


@pytest.mark.parametrize("verify", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("rhs", list(RHS))
@pytest.mark.parametrize("path", list(PATHS))
def test_solve(cuda, path, rhs, prec, verify):
    make, kw = PATHS[path]
    op = make(cuda)
    op.set_shifts([0.0, 0.1, 1.0])
    b = RHS[rhs](W.gaussian_rhs(op.n, 642))
    _broke_down(*op.solve(b, tol=1e-8, prec=prec, verify=verify, check=False, **kw))
    op.close()


@pytest.mark.parametrize("verify", [True, False])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("rhs", list(RHS))
def test_solve_real(cuda, rhs, prec, verify):
    # in single precision the scaled entries are infinite themselves
    op = _grid(cuda)
    op.set_shifts([0.01, 0.1, 1.0])
    b = RHS[rhs](np.random.default_rng(643).standard_normal(op.n))
    _broke_down(*op.solve_real(b, tol=1e-8, prec=prec, verify=verify, check=False))
    op.close()
