"""The FP64 GP likelihood keeps its roundings.  Where sigma_f^2 / sigma_n^2 is large the covariance's
condition number turns another order of a sum, or another rounding of a root or an exponential,
into 1e-9 of log L, more than any bar against another implementation can see.  So the values are
pinned, bit for bit, to recorded ones (the evaluation and the chains of two iterations), at a
ragged single block pair, ragged and full tiles and the largest size."""
import numpy as np
import pytest
from conftest import read_golden

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def recorded():
    rows = read_golden("gp_ill_conditioned.txt")
    f = lambda r: [float.fromhex(v) for v in r]  # noqa: E731
    data = np.array([f(r[1:]) for r in rows if r[0] == "data"])
    points = {}
    live = {}
    for r in rows:
        if r[0] == "point":
            points.setdefault(int(r[1]), []).append(f(r[2:]))
        if r[0] == "live":
            live.setdefault(int(r[1]), []).append(float.fromhex(r[2]))
    return data, points, live


@pytest.mark.parametrize("n", [23, 100, 129, 256])
def test_values_are_the_recorded_ones(recorded, n):
    from paper_2601_23252_amd import nss, problems as G
    data, points, live = recorded
    prob = dict(G.gp_problem(4, n=n, m=40, k=10), gp_x=data[:n, :2].copy(), gp_y=data[:n, 2].copy())
    R = nss.NSRun(prob, m=40, k=10, p=4, seed=5)
    P = np.array(points[n])
    assert np.array_equal(R.eval_loglik(P[:, :6], "fp64"), P[:, 6])
    R.step()
    R.step()
    s = R.state()
    R.close()
    assert np.array_equal(s["logL"][s["perm"]], np.array(live[n]))
