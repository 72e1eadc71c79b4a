"""GPU: the batched CG (systems that share an operator) on each storage, against dense solves.

Right-hand sides per shift with repeated shifts go to the batched CG.  It takes the systems
still iterating in groups (two on the links, five on the stored matrix), so counts around
those sizes and around the most systems of one call are tried, on a lattice whose volume
leaves a partial block and one that fills whole blocks; the shifts span three decades, so
that systems leave the list at different iterations.

Tolerance: |x - x*| <= cond |r| / |A|, cond(A + s) <= 3.6 / 0.01 here and |r| <= 1e-12 |b|:
4e-10 relative, doubled.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(4, 4, 4, 4), (3, 5, 4, 3)])
def lattice(request):
    dims = request.param
    links = W.random_su3_links(dims, 501)
    n = 3 * W.lattice_volume(dims)
    rowptr, col, vals = W.staggered_csr(links, dims, 0.1)
    m = np.zeros((n, n), complex)
    m[np.repeat(np.arange(n), np.diff(rowptr)), col] = vals
    return dict(dims=dims, links=links, n=n, csr=(rowptr, col, vals), a=m.conj().T @ m)


@pytest.mark.parametrize("storage", ["links", "sell", "csr"])
@pytest.mark.parametrize("ns", [2, 3, 5, 6, 11, 16, 17])
def test_systems_and_groups(lattice, cuda, ns, storage):
    from paper_1102_2143_amd import Operator
    p = lattice
    print(f"[gpu] batched CG dims={p['dims']} ns={ns} {storage}", flush=True)
    sigma = np.resize([1e-3, 1e-3, 1.0, 0.03, 0.3, 1e-3, 0.1], ns)
    b = W.gaussian_rhs(p["n"], 502, ns)
    if storage == "links":
        op = Operator.staggered(p["links"], p["dims"], 0.1, device=cuda)
    else:
        op = Operator(*p["csr"], p["n"], kind="mhm", device=cuda)
    op.set_shifts(sigma)
    x, info = op.solve_multi_rhs(b, tol=1e-12, format="auto" if storage == "links" else storage)
    x = x.cpu().numpy()
    assert info["status"] == "ok" and info["iters"] == 0
    for k in range(ns):
        ref = np.linalg.solve(p["a"] + sigma[k] * np.eye(p["n"]), b[k])
        assert np.linalg.norm(x[k] - ref) <= 8e-10 * np.linalg.norm(ref), k
    op.close()
