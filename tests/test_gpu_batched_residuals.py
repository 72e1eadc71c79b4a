"""GPU: the residuals a batched solve reports are those of the matrix itself.

The batch verifies operators made from links with the kernels that read links, so a wrong copy of
them would not show in its own figures: here they are compared with residuals formed on the host
from the CSR that the links define.  Both round by some eps |A| |x| <= 1e-12 of b, a hundredth
of the residuals' 1e-10.
"""
import numpy as np
import pytest

import oracle as O
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("scale", [1.0, 1.0 + 3e-13, 1.05])
def test_reported_residuals(cuda, scale, prec):
    from paper_1102_2143_amd import Operator, solve_batched
    dims, sigma = [(4, 4, 4, 4), (3, 5, 4, 7)], [0.3, 0.01, 0.0]
    links = [scale * W.random_su3_links(d, 691 + i) for i, d in enumerate(dims)]
    ops = [Operator.staggered(l, d, 0.1, device=cuda) for l, d in zip(links, dims)]
    bs = [W.gaussian_rhs(op.n, 695, 3) for op in ops]
    for op in ops:
        op.set_shifts(sigma)
    xs, infos, status = solve_batched(ops, bs, tol=1e-10, prec=prec)
    assert status == "ok"
    for i, op in enumerate(ops):
        csr = W.staggered_csr(links[i], dims[i], 0.1)
        for q in range(3):
            x, b = xs[i][q].cpu().numpy(), bs[i][q]
            host = [np.linalg.norm(b - O.shifted_apply("mhm", *csr, op.n)(x[k], s)) / np.linalg.norm(b)
                    for k, s in enumerate(sigma)]
            assert np.allclose(infos[3 * i + q]["true_rel_res"], host, rtol=0.02, atol=1e-12)
        op.close()
