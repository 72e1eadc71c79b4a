"""GPU: batches in which some systems have a few eigenvalues far above the rest (see
test_gpu_stiff.py), beside ordinary ones: those take their directions up, the others go on without.

Every right-hand side ends within the oracle's steps, a quarter and ten more (in complex64 as many
again, as there), meets the tolerance by its true residual formed on the host after the refinement,
and an indefinite system in between is a breakdown of its own.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W
from test_gpu_stiff import grid, stiff_links

pytestmark = pytest.mark.gpu

TOL = 1e-10
SIGMA = [0.1, 0.0, 1.0]


def _systems(cuda, penalty):
    """(operator, kind, csr) of each: an ordinary grid, the grid with the penalty (A given), links
    with one far above the others, the grid as M with the penalty's root."""
    from paper_1102_2143_amd import Operator
    out = []
    for p in (0.0, penalty):
        csr = grid(24, 1e-2, p)
        out.append((Operator(*csr, kind="herm", device=cuda), "herm", csr))
    dims = (4, 4, 4, 5)
    links = stiff_links(dims, np.sqrt(penalty))
    out.append((Operator.staggered(links, dims, 0.1, device=cuda), "mhm",
                (*W.staggered_csr(links, dims, 0.1), 3 * W.lattice_volume(dims))))
    csr = grid(12, 0.3, np.sqrt(penalty))
    out.append((Operator(*csr, kind="mhm", device=cuda), "mhm", csr))
    return out


@pytest.mark.parametrize("fmt", ["auto", "csr"])
@pytest.mark.parametrize("prec,more", [("fp64", 1.25), ("mixed", 2.0)])
@pytest.mark.parametrize("nrhs,steps,poll", [(1, 8, 16), (3, 3, 10), (4, 1, 5)])
@pytest.mark.parametrize("penalty", [1.0, 1e4, 1e8])
def test_batch(cuda, penalty, nrhs, steps, poll, prec, more, fmt):
    from paper_1102_2143_amd import solve_batched
    systems = _systems(cuda, penalty)
    for op, _, _ in systems:
        op.set_shifts(SIGMA)
    bs = [W.gaussian_rhs(op.n, 731 + i, nrhs) for i, (op, _, _) in enumerate(systems)]
    xs, infos, status = solve_batched([s[0] for s in systems], bs, tol=TOL, prec=prec, format=fmt,
                                      update_steps=steps, poll_every=poll)
    assert status == "ok"
    for i, (op, kind, csr) in enumerate(systems):
        ap = O.shifted_apply(kind, *csr)
        for q in range(nrhs):
            info = infos[i * nrhs + q]
            ref = O.cg_m(ap, bs[i][q], np.array(SIGMA), tol=TOL)
            print(f"[gpu] batch penalty={penalty:g} {prec} {fmt} system {i} rhs {q} "
                  f"iters={info['iters']} oracle={ref['iters']} refine={info['refine_iters']}", flush=True)
            assert info["iters"] <= more * ref["iters"] + 10
            x = xs[i][q].cpu().numpy()
            for k, s in enumerate(SIGMA):
                r = bs[i][q] - ap(x[k], s)
                assert np.linalg.norm(r) <= 1.05 * TOL * np.linalg.norm(bs[i][q]), (i, q, k)
        op.close()


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("penalty", [0.0, 1e8])
def test_not_positive_definite(cuda, penalty, prec):
    from paper_1102_2143_amd import Operator, solve_batched
    good, bad = grid(16, 1e-2, penalty), grid(15, 1e-3, penalty)
    ops = [Operator(*c, kind="herm", device=cuda) for c in (good, bad)]
    ops[0].set_shifts([0.0, 0.1])
    ops[1].set_shifts([-0.5, 0.1])
    bs = [W.gaussian_rhs(op.n, 741 + i, 2) for i, op in enumerate(ops)]
    xs, _, status = solve_batched(ops, bs, tol=1e-8, prec=prec, check=False)
    assert status == "breakdown"
    ap = O.shifted_apply("herm", *good)
    for q in range(2):
        x = xs[0][q].cpu().numpy()
        for k, s in enumerate((0.0, 0.1)):
            r = bs[0][q] - ap(x[k], s)
            assert np.linalg.norm(r) <= 1.05e-8 * np.linalg.norm(bs[0][q])
    for op in ops:
        op.close()
