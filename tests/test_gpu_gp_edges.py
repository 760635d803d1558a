"""The GP likelihood at the edges of its 16-row blocks and of the tiles per wave, against the FP64
oracle, with the bar of the other sizes: |d log L| <= 1e-9 |log L| + 1e-14 kappa (1 + |log L| / n),
kappa = n (sigma_f^2 + sigma_n^2) / sigma_n^2, and the same set of breakdowns."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 15, 16, 17, 31, 32, 33, 64, 65, 112, 113, 128, 129, 240, 241, 255])
def test_gp_loglik_at_block_edges(oracle_lib, n):
    from paper_2601_23252_amd import nss, problems as G
    prob = G.gp_problem(4, n=n, m=64, k=16)
    rng = np.random.default_rng(n)
    X = np.vstack([rng.uniform(prob["prior_a"], prob["prior_b"], (24, 6)),
                   np.log(np.array(G.GP_THETA_TRUE)) + 0.3 * rng.standard_normal((12, 6))])
    R = nss.NSRun(prob, m=64, k=16, p=1, seed=0)
    g = R.eval_loglik(X, "fp64")
    R.close()
    o = oracle_lib.Problem(prob).loglik(X)
    assert np.array_equal(np.isfinite(g), np.isfinite(o))
    f = np.isfinite(o)
    th = np.exp(X[f])
    kappa = n * (th[:, 0] ** 2 + th[:, 5] ** 2) / th[:, 5] ** 2
    tol = 1e-9 * np.abs(o[f]) + 1e-14 * kappa * (1 + np.abs(o[f]) / n)
    assert np.all(np.abs(g[f] - o[f]) <= tol), np.max(np.abs(g[f] - o[f]) / tol)
