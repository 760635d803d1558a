"""The geometric uncertainty at the edges of its chunks (512 deaths, 8 a lane) and past 64 replicas a
group (where the next chunk's first shrinkage is drawn anew), against the FP64 oracle on the run's
own dead record.  The bars are those of the full runs' comparison: prefix sums of |log X| in another
order, the mean over R values of size |log w|, and a few ulp of t t' over 1 - t t' >= ~1/n."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def N():
    from paper_2601_23252_amd import nss
    nss.load()
    return nss


@pytest.mark.parametrize("m,R", [(3, 1), (7, 65), (8, 100), (9, 3), (511, 20), (512, 20), (513, 20),
                                 (520, 9), (1023, 100), (1024, 100), (1025, 100), (2500, 65535)])
def test_chunk_edges_and_replica_groups(N, oracle_lib, m, R):
    """Right after initialisation a run of m points has m deaths."""
    from paper_2601_23252_amd import problems as G
    prob = G.gaussian_problem(3, np.zeros(3), 0.09 * np.eye(3))
    run = N.NSRun(prob, m=m, k=max(1, m // 3), p=1, seed=m)
    s = run.state()
    dead, fin = run.dead(), np.sort(s["logL"][s["perm"][run.k:]])
    L = np.concatenate([dead, fin])
    assert len(L) == m
    g = run.geom(R=R, beta=1.0, seed=5, run_id=2)
    run.close()
    z, lw, ess = oracle_lib.geom(dead, fin, m, max(1, m // 3), R, 1.0, 5, 2)
    scale = 1.0 + np.abs(lw - L) + np.log(2 * m)
    assert np.all(np.abs(g["logw_mean"] - lw) <= 1e-12 * scale + EPS * R * np.abs(lw) + 8 * EPS * m)
    assert np.all(np.abs(g["logz"] - z) <= 1e-12 * scale.max() + EPS * np.abs(lw).max() + 8 * EPS * m)
    assert abs(g["ess"] - ess) <= 1e-10 * ess
