"""GPU: update_steps of the BiCGStab-M solve is the number of steps folded into one application, up
to four: every number gives the oracle's iterates, 1 to 4 round differently, and larger ones act as 4.

After nine steps 1e-11, as the stops around an application of four steps."""
import numpy as np
import pytest

import oracle as O
from test_gpu_bicgstab_steps import _problem, _rel, _solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fmt", ["sell", "csr"])
def test_update_steps(cuda, fmt):
    p = _problem((7, 6, 5), 5)
    ref = O.bicgstab_m(p["apply"], p["b"], p["sigma"], tol=0.0, max_iter=9)
    x = {k: _solve(p, cuda, tol=1e-30, max_iter=9, format=fmt, update_steps=k)[0] for k in (1, 2, 3, 4, 8)}
    for k in x:
        assert _rel(x[k], ref["x"]) <= 1e-11, k
    assert np.array_equal(x[8], x[4])
    for k in (1, 2, 3):
        assert not np.array_equal(x[k], x[k + 1]), k
