"""GPU: iters_fp64 of a batched mixed solve where the first right-hand side has nothing to do: the
count is the system's, whichever of its right-hand sides still iterate at the switch."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zero", [0, 1, 2])
def test_fp64_iterations(cuda, zero):
    from paper_1102_2143_amd import Operator, solve_batched
    rowptr, col, vals = W.laplacian7_csr((7, 6, 5), 751)
    op = Operator(rowptr, col, vals, 210, kind="herm", device=cuda)
    op.set_shifts([0.0, 0.1])
    b = W.gaussian_rhs(210, 752, 3)
    b[zero] = 0.0
    _, infos, status = solve_batched([op], [b], tol=1e-10, prec="mixed")
    assert status == "ok"
    assert infos[zero]["iters"] == 0
    for q in range(3):
        if q != zero:
            assert 0 < infos[q]["iters_fp64"] < infos[q]["iters"], infos[q]
    assert np.isfinite([i["alg_bytes"] for i in infos]).all()
    op.close()
