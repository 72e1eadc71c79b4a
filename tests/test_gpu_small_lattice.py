"""GPU: lattices that one workgroup holds, several iterations to a launch, against the oracle.

Volumes that fill the workgroup's 256 sites, that leave lanes idle, and one just above (the
pair of kernels); SU(3) links (two rows read) and links off SU(3) (nine values).  A launch
ends where steps are applied, the host polls or an update falls due, so these are varied
against each other and against where the sequence stops.

Tolerances: after at most 20 steps the iterates agree to rounding, 20 steps of a sequence whose
roundings grow by at most the condition 700: 20 * 700 * 1.1e-16 * 4 = 6e-12.  To a tolerance
of 1e-10, |x - x*| <= cond |r| / |A|, cond(A + s) <= 8.5 / 0.01: 8.5e-8.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

DIMS = [(3, 3, 3, 3), (3, 3, 4, 7), (4, 4, 4, 4), (3, 3, 3, 10)]


def _problem(dims, scale, cuda, ns=5):
    from paper_1102_2143_amd import Operator
    links = scale * W.random_su3_links(dims, 631)
    n = 3 * W.lattice_volume(dims)
    op = Operator.staggered(links, dims, 0.1, device=cuda)
    sigma = np.concatenate([[0.3, 0.0], W.logspace_shifts(1e-3, 1.0, ns - 2)])
    op.set_shifts(sigma)
    ap = O.shifted_apply("mhm", *W.staggered_csr(links, dims, 0.1), n)
    return op, W.gaussian_rhs(n, 632), sigma, ap


@pytest.mark.parametrize("dims", DIMS)
@pytest.mark.parametrize("limit,steps,poll", [(1, 8, 16), (5, 3, 16), (8, 8, 16), (9, 8, 3), (20, 8, 16)])
def test_first_steps(cuda, dims, limit, steps, poll):
    print(f"[gpu] small lattice dims={dims} limit={limit} steps={steps} poll={poll}", flush=True)
    op, b, sigma, ap = _problem(dims, 1.0, cuda)
    x, info = op.solve(b, tol=1e-13, max_iter=limit, refine=False, update_steps=steps, poll_every=poll)
    ref = O.cg_m(ap, b, sigma, tol=1e-13, max_iter=limit)
    assert info["iters"] == limit
    err = np.linalg.norm(x.cpu().numpy() - ref["x"], axis=1) / np.linalg.norm(ref["x"], axis=1)
    assert np.all(err <= 6e-12), err
    op.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("scale,ns", [(1.0, 5), (1.1, 33)])
@pytest.mark.parametrize("dims", DIMS)
def test_solve(cuda, dims, scale, ns, prec):
    print(f"[gpu] small lattice dims={dims} scale={scale} ns={ns} {prec}", flush=True)
    op, b, sigma, ap = _problem(dims, scale, cuda, ns)
    ref = O.cg_m(ap, b, sigma, tol=1e-13)
    for kw in (dict(), dict(update_steps=3, poll_every=10, reliable_every=15), dict(timing=1)):
        x, info = op.solve(b, tol=1e-10, prec=prec, **kw)
        assert info["status"] == "ok" and np.all(info["true_rel_res"] <= 1e-10)
        assert (info["n_reliable"] > 0) == (prec == "mixed")
        err = np.linalg.norm(x.cpu().numpy() - ref["x"], axis=1) / np.linalg.norm(ref["x"], axis=1)
        assert np.all(err <= 8.5e-8), (kw, err)
    op.close()


def test_no_steps(cuda):
    # a right-hand side of zero, and a limit of no steps: x = 0 without one
    op, b, sigma, _ = _problem((4, 4, 4, 4), 1.0, cuda)
    for rhs, kw in ((np.zeros_like(b), {}), (b, dict(max_iter=0, refine=False))):
        x, info = op.solve(rhs, tol=1e-10, **kw)
        assert info["iters"] == 0 and not bool(x.abs().any())
    op.close()
