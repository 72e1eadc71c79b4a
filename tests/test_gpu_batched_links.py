"""GPU: batched multishift solves of operators made from links, against dense solves.

A wave takes 64 sites of one right-hand side and a workgroup's four waves 64, 128 or 256
sites of four, two or one of them, so lattices below one wave, with a partial block and with
several blocks are tried for each padding of the right-hand sides (three pad to four); SU(3)
links (two rows read) beside links that are not (three rows), and a stored matrix between
them.  The composed steps are applied every update_steps launches and by the last of
poll_every, so counts that divide and that do not are tried; in mixed precision every system
changes precision at one of these applications, and a reliable update follows the last.

Tolerance: |x - x*| / |x*| <= cond |r| / |b|, cond(A + s) <= 6.95 / 0.01 for the lattices
(6.93 + m^2 is the largest eigenvalue of these links' A) and less for the stored matrix, |r|
<= 1e-10 |b|: 7.0e-8.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

DIMS = [(3, 3, 4, 3), (4, 4, 4, 4), (3, 5, 4, 7)]


def _dense(rowptr, col, vals, n):
    m = np.zeros((n, n), complex)
    m[np.repeat(np.arange(n), np.diff(rowptr)), col] = vals
    return m


@pytest.fixture(scope="module")
def systems():
    out = []
    for i, dims in enumerate(DIMS):
        links = W.random_su3_links(dims, 601 + i)
        if i == 1:  # no third row to rebuild from the other two
            links = links * (0.9 + 0.1 * np.random.default_rng(7).random(links.shape[:2])[..., None, None])
        n = 3 * W.lattice_volume(dims)
        m = _dense(*W.staggered_csr(links, dims, 0.1), n)
        out.append(dict(links=links, dims=dims, n=n, a=m.conj().T @ m))
    rowptr, col, vals = W.laplacian7_csr((7, 6, 5), 611)
    out.insert(1, dict(csr=(rowptr, col, vals), n=210, a=_dense(rowptr, col, vals, 210)))
    return out


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("nrhs,steps,poll", [(1, 8, 16), (2, 3, 10), (3, 1, 16), (4, 8, 5)])
def test_links_in_a_batch(systems, cuda, nrhs, steps, poll, prec):
    from paper_1102_2143_amd import Operator, solve_batched
    print(f"[gpu] batch on links nrhs={nrhs} steps={steps} poll={poll} {prec}", flush=True)
    ops, bs = [], []
    for i, p in enumerate(systems):
        op = (Operator(*p["csr"], p["n"], kind="herm", device=cuda) if "csr" in p
              else Operator.staggered(p["links"], p["dims"], 0.1, device=cuda))
        op.set_shifts(np.array([0.3, 0.0, 1.0, 0.03][: 4 - i % 2]))
        ops.append(op)
        bs.append(W.gaussian_rhs(p["n"], 620 + i, 4)[:max(1, nrhs - i % 2)])
    xs, infos, status = solve_batched(ops, bs, tol=1e-10, prec=prec, update_steps=steps,
                                      poll_every=poll, reliable_every=20)
    assert status == "ok", [i["status"] for i in infos]
    t = 0
    for i, p in enumerate(systems):
        x = xs[i].cpu().numpy()
        for q in range(len(bs[i])):
            assert np.all(infos[t]["true_rel_res"] <= 1e-10), (i, q)
            t += 1
            for k, s in enumerate([0.3, 0.0, 1.0, 0.03][: 4 - i % 2]):
                ref = np.linalg.solve(p["a"] + s * np.eye(p["n"]), bs[i][q])
                assert np.linalg.norm(x[q][k] - ref) <= 7.2e-8 * np.linalg.norm(ref), (i, q, k)
    for op in ops:
        op.close()
