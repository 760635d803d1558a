"""The GP likelihood at length scales far below the inputs' spacing, where the kernel's exponent is
-1e35 to -1e89 and every entry off the diagonal is exactly zero: log L is finite and, as the
covariance is then a multiple of the identity, the oracle's to rounding.  FP64: 1e-12 relative (64
equal pivots, a logarithm and a sum of squares).  FP32: the pivot's rounding, 6e-8, moves half of
64 equal logarithms by 2e-6; the quadratic form is refined in FP64: 1e-7 |log L| is five times
that."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("coord", [1, 2, 3])
@pytest.mark.parametrize("value", [-40.0, -50.0, -100.0])
def test_tiny_length_scales(oracle_lib, coord, value):
    from paper_2601_23252_amd import nss, problems as G
    prob = G.gp_problem(4, n=64, m=40, k=10)
    u = np.array([[0.0, 0.7, 1.0, 0.0, 1.0, -2.0]])
    u[0, coord] = value
    R = nss.NSRun(prob, m=40, k=10, p=1, seed=0)
    g, f = R.eval_loglik(u, "fp64")[0], R.eval_loglik(u, "fp32")[0]
    R.close()
    o = oracle_lib.Problem(prob).loglik(u)[0]
    assert np.isfinite(o)
    assert abs(g - o) <= 1e-12 * abs(o), (g, o)
    assert abs(f - o) <= 1e-7 * abs(o), (f, o)
