"""GPU: the operator applied on its own, on each storage it reads, against the oracle's product.

FP64 products read the links from 16384 sites on (two rows per link when they are SU(3) to
1e-14, else all nine values; marching along t where the lattice allows it and each wave
gets a run), the sliced copy from 16384 rows on, else the CSR.  Each is tried at the sizes
where it can go wrong: a partial last block of 64 sites, the smallest size of a path and
the one below it, a marched lattice.  Input and output may be the same buffer.

Tolerance: a product is two sums of 25 terms, each within 27 u of its terms' moduli (u =
1.1e-16), and the terms' moduli sum to at most 5 times the rows' norm here: 2 * 27 * 5 u =
3e-14 bounds the relative error in the 2-norm; a rebuilt third row adds at most the 1e-14
that its use is limited to, twice.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("scale", [1.0, 1.25])  # SU(3) links, and links off SU(3)
@pytest.mark.parametrize("dims", [(8, 8, 16, 16), (9, 12, 13, 12),
                                  (3, 3, 43, 43), (32, 32, 16, 32)])
def test_links(cuda, dims, scale):
    from paper_1102_2143_amd import Operator
    if scale != 1.0 and W.lattice_volume(dims) > 100_000:
        pytest.skip("the march reads two-row links only")
    print(f"[gpu] apply on links dims={dims} scale={scale}", flush=True)
    links = scale * W.random_su3_links(dims, 401)
    n = 3 * W.lattice_volume(dims)
    v = W.gaussian_rhs(n, 402)
    ref = O.shifted_apply("mhm", *W.staggered_csr(links, dims, 0.07), n)(v, 0.3)
    op = Operator.staggered(links, dims, 0.07, device=cuda)
    assert op.storage()["two_rows"] == (scale == 1.0)
    assert _rel(op.apply(v, shift=0.3).cpu().numpy(), ref) <= 5e-14
    op.close()


@pytest.mark.parametrize("kind,prec", [("mhm", "fp64"), ("herm", "fp64"), ("herm", "mixed")])
@pytest.mark.parametrize("n", [16383, 16384, 16385, 30000])
def test_stored_matrix_and_in_place(cuda, n, kind, prec):
    import torch
    from paper_1102_2143_amd import Operator
    print(f"[gpu] apply on the stored matrix n={n} {kind} {prec}", flush=True)
    rowptr, col, vals = W.poisson5pt_csr(n // 3 if n % 3 == 0 else n, 3 if n % 3 == 0 else 1)
    n = rowptr.size - 1
    vals = vals * (1.0 + np.random.default_rng(5).uniform(0.0, 0.5, vals.size))
    v = W.gaussian_rhs(n, 403)
    ref = O.shifted_apply(kind, rowptr, col, vals, n)(v, 0.5)
    op = Operator(rowptr, col, vals, n, kind=kind, device=cuda)
    got = op.apply(v, shift=0.5, prec=prec)
    # complex64: 2 ** 29 times the unit, on sums of 5 terms
    assert _rel(got.cpu().numpy(), ref) <= (3e-14 if prec == "fp64" else 2e-6)
    buf = torch.from_numpy(v).to(cuda)
    op.apply_noalloc(buf, buf, shift=0.5, prec=prec)
    torch.cuda.synchronize()
    assert torch.equal(buf, got)
    op.close()
