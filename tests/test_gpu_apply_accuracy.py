"""GPU: the FP64 product is as accurate from the links and the sliced copy as from the CSR.

Against the product in extended precision.  The CSR's eight lanes add three entries each and
then in pairs: a sum of 25 terms carries the rounding of a leaf of three complex terms and of
three levels above it, twice, with the shift: 1.37e-16 of the result in the 2-norm over lattices
of 32768 sites and more; one chain of 24 terms carries 2.6e-16, and a third link row rebuilt
from two 3.4e-16.  The bar lies between, about a tenth above the first.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

BAR = 1.5e-16


def _exact(rowptr, col, vals, v, shift):
    n = rowptr.size - 1
    vals, v = vals.astype(np.clongdouble), v.astype(np.clongdouble)
    u = np.add.reduceat(vals * v[col], rowptr[:-1])
    row = np.repeat(np.arange(n), np.diff(rowptr))
    order = np.argsort(col, kind="stable")
    first = np.concatenate([[0], np.cumsum(np.bincount(col, minlength=n))[:-1]])
    return np.add.reduceat((np.conj(vals) * u[row])[order], first) + shift * v


@pytest.mark.parametrize("source", ["links", "sliced"])
@pytest.mark.parametrize("scale", [1.0, 1.0 + 2e-13, 1.25])  # SU(3), near it and off it
@pytest.mark.parametrize("dims", [(16, 16, 16, 8), (12, 10, 14, 11), (16, 16, 16, 16)])
def test_product(cuda, dims, scale, source):
    from paper_1102_2143_amd import Operator
    print(f"[gpu] product accuracy dims={dims} scale={scale} {source}", flush=True)
    links = scale * W.random_su3_links(dims, 671)
    csr = W.staggered_csr(links, dims, 0.1)
    n = 3 * W.lattice_volume(dims)
    v = W.gaussian_rhs(n, 672)
    if source == "links":
        op = Operator.staggered(links, dims, 0.1, device=cuda)
    else:
        op = Operator(*csr, n, kind="mhm", device=cuda)
        assert op.storage()["sell"]
    ref = _exact(*csr, v, 0.3)
    err = (op.apply(v, shift=0.3).cpu().numpy() - ref).astype(complex)
    assert np.linalg.norm(err) <= BAR * np.linalg.norm(ref.astype(complex))
    op.close()
