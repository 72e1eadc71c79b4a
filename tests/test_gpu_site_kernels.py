"""GPU: the links' kernels with one site per lane, on lattices that a default grid would give to
the kernels with a direction per wave: a capped grid leaves several blocks of 64 sites to a wave.

A partial last block, the lattice's order (planes of whole blocks), and marches in columns of 2, 4,
8 and 16 t-slices (the largest power of two that divides L_t) with at least four blocks to each
wave of the capped grid; SU(3) links and nine values.  FP64 against the oracle's iterates at
1e-10 and iterations, mixed at 1e-12, to 1e-8 as the other parity tests.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu

CASES = [((5, 5, 5, 7), 8), ((3, 4, 7, 9), 8), ((8, 8, 8, 8), 8), ((8, 8, 16, 10), 8),
         ((8, 8, 16, 12), 8), ((8, 8, 8, 24), 8), ((8, 8, 8, 32), 16)]


@pytest.mark.parametrize("scale", [1.0, 1.02])
@pytest.mark.parametrize("dims,grid", CASES)
def test_site_kernels(cuda, dims, grid, scale):
    from paper_1102_2143_amd import Operator
    blocks = -(-W.lattice_volume(dims) // 64)
    assert blocks > grid  # else a direction per wave
    mass = 0.1
    links = scale * W.random_su3_links(dims, 701)
    csr, n = W.staggered_csr(links, dims, mass), 3 * W.lattice_volume(dims)
    sigma = np.concatenate([[0.2], W.logspace_shifts(1e-4, 1.0, 4)])
    b = W.gaussian_rhs(n, 702)
    ap = O.shifted_apply("mhm", *csr, n)
    op = Operator.staggered(links, dims, mass, device=cuda)
    op.set_shifts(sigma)
    for prec, tol in (("fp64", 1e-10), ("mixed", 1e-12)):
        print(f"[gpu] site kernels dims={dims} grid={grid} scale={scale} {prec}", flush=True)
        x, info = op.solve(b, tol=tol, prec=prec, max_grid=grid)
        assert info["status"] == "ok" and np.all(info["true_rel_res"] <= tol)
        ref = O.cg_m(ap, b, sigma, tol=tol if prec == "fp64" else 1e-13)
        if prec == "fp64":
            assert abs(info["iters"] - ref["iters"]) <= 2
        err = np.linalg.norm(x.cpu().numpy() - ref["x"], axis=1) / np.linalg.norm(ref["x"], axis=1)
        assert np.all(err <= 1e-8), err
    op.close()
