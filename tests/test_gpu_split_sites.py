"""GPU: the links' kernels with a wave for each direction, and with a site per lane, against the oracle.

A lattice of at most max_grid (default 1024) blocks of 64 sites takes the first form; a
small max_grid takes the second on the same lattice.  Tried on volumes of one site block,
of a partial last block and of exactly max_grid blocks, with SU(3) links (two rows) and
links off SU(3) (nine values), FP64 and mixed, and with steps applied one by one.

Tolerance: the solves run to tol 1e-10 (mixed 1e-11 against the oracle at 1e-12); |dx|/|x| <=
cond * tol with cond <= 4 / 0.0101 here.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("scale", [1.0, 1.1])
@pytest.mark.parametrize("dims,grid", [((4, 4, 4, 4), 0), ((3, 5, 4, 3), 0), ((3, 5, 7, 9), 0),
                                       ((3, 5, 7, 9), 8), ((4, 8, 4, 4), 8), ((4, 8, 4, 8), 8)])
def test_solve(cuda, dims, grid, scale, prec):
    from paper_1102_2143_amd import Operator
    print(f"[gpu] split sites dims={dims} grid={grid} scale={scale} {prec}", flush=True)
    links = scale * W.random_su3_links(dims, 601)
    n = 3 * W.lattice_volume(dims)
    b = W.gaussian_rhs(n, 602)
    sigma = W.logspace_shifts(1e-4, 1.0, 5)
    ap = O.shifted_apply("mhm", *W.staggered_csr(links, dims, 0.1), n)
    tol = 1e-10 if prec == "fp64" else 1e-11
    ref = O.cg_m(ap, b, sigma, tol=tol if prec == "fp64" else 1e-12)
    op = Operator.staggered(links, dims, 0.1, device=cuda)
    op.set_shifts(sigma)
    for steps in (8, 1):
        x, info = op.solve(b, tol=tol, prec=prec, max_grid=grid, update_steps=steps)
        assert info["status"] == "ok"
        err = np.linalg.norm(x.cpu().numpy() - ref["x"], axis=1) / np.linalg.norm(ref["x"], axis=1)
        assert np.all(err <= 5e-8), (steps, err)
        if prec == "fp64":
            assert abs(info["iters"] - ref["iters"]) <= 2
    op.close()
