"""The kernels beside the chains at the edges of their layouts, through the C ABI: delete-k's
register sort around its powers of two and its elements per thread (64, 1024, 2048 and 4096
points), with ties; the whitening factor around its 16-column blocks and its 48 rows per wave."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def N():
    from paper_2601_23252_amd import nss
    nss.load()
    return nss


@pytest.mark.parametrize("m", [2, 3, 63, 64, 65, 127, 129, 1000, 1024, 1025, 2048, 2049, 4096,
                               4097, 8192])
def test_delete_k_order_with_ties(N, m):
    """perm is the ascending (logL, index) order of an injected live set with many equal values,
    -inf among them; L* its k-th value."""
    from paper_2601_23252_amd import problems as G
    prob = G.gaussian_problem(3, np.zeros(3), np.eye(3))
    k = max(1, m // 3)
    r = N.NSRun(prob, m=m, k=k, p=2, seed=1)
    s = r.state()
    rng = np.random.default_rng(m)
    L = np.round(rng.normal(size=m) * 8.0) / 4.0
    L[rng.random(m) < 0.02] = -np.inf
    L[rng.integers(m)] = L[np.isfinite(L)].max(initial=0.0) + 1.0   # something above L*
    r.set_state(s["x"], L, s["logZ"], s["logX"], s["M"], s["iter"])
    got = r.state()
    want = np.lexsort((np.arange(m), L))
    assert np.array_equal(got["perm"], want)
    assert got["Lstar"] == L[want[k - 1]]
    r.close()


@pytest.mark.parametrize("d", [1, 15, 16, 17, 31, 33, 63, 64, 65, 80, 97, 112, 127, 128])
@pytest.mark.parametrize("diagonal", [False, True])
def test_whitening_factor(N, d, diagonal):
    """L L^T equals the survivors' population covariance (numpy) plus the jitter, relative to the
    variances: both sides round at about 1e-16 times the number of points and columns summed."""
    from paper_2601_23252_amd import problems as G
    prob = G.gaussian_problem(d, np.zeros(d), 0.04 * np.eye(d))
    m, k = 400, 130
    r = N.NSRun(prob, m=m, k=k, p=1, seed=d, diagonal_metric=diagonal)
    s = r.state()
    pts = s["x"][s["perm"][k:]]
    r.step()
    L = r.state()["Lsig"]
    C = np.cov(pts.T, bias=True).reshape(d, d)
    C = np.diag(np.diag(C)) if diagonal else C
    C = C + 1e-12 * np.trace(C) / d * np.eye(d)
    sd = np.sqrt(np.diag(C))
    assert np.array_equal(L, np.tril(L))
    assert np.abs((L @ L.T - C) / np.outer(sd, sd)).max() < 1e-12
    assert r.stats()["whiten_fallbacks"] == 0
    r.close()


def test_singular_covariance_falls_back_to_the_variances(N):
    """Survivors on a line: where rounding leaves a pivot that is not positive the factor is the
    diagonal one, and counted; else the jitter carried the factorisation."""
    from paper_2601_23252_amd import problems as G
    d, m, k = 40, 60, 20
    prob = G.gaussian_problem(d, np.zeros(d), np.eye(d), "box", -1e6, 1e6)
    r = N.NSRun(prob, m=m, k=k, p=1, seed=3)
    s = r.state()
    rng = np.random.default_rng(0)
    x = 1e5 * rng.normal(size=(m, 1)) * np.ones((1, d))   # rank one
    x[:, 1::2] *= -1.0
    L = -np.arange(m, dtype=float)
    r.set_state(x, L, s["logZ"], s["logX"], s["M"], s["iter"])
    r.step()
    st = r.state()
    if r.stats()["whiten_fallbacks"]:
        off = st["Lsig"] - np.diag(np.diag(st["Lsig"]))
        assert np.all(off == 0.0)
        surv = x[np.argsort(L, kind="stable")[k:]]
        assert np.allclose(np.diag(st["Lsig"]), surv.std(axis=0), rtol=1e-9)
    else:   # the jitter carried it: the factor is finite and reproduces the covariance
        assert np.all(np.isfinite(st["Lsig"]))
    r.close()


@pytest.mark.parametrize("d", [24, 33, 64, 100, 128])
def test_whitening_factor_of_few_survivors(N, d):
    """20 survivors in d > 20 dimensions: the covariance is singular but for the jitter (1e-12 of the
    mean variance), which the factor still holds: no fallback, and L L^T equals the covariance to the
    rounding of 20 + d summands."""
    from paper_2601_23252_amd import problems as G
    prob = G.gaussian_problem(d, np.zeros(d), 0.04 * np.eye(d))
    r = N.NSRun(prob, m=40, k=20, p=1, seed=d)
    s = r.state()
    pts = s["x"][s["perm"][20:]]
    r.step()
    L = r.state()["Lsig"]
    C = np.cov(pts.T, bias=True).reshape(d, d)
    C = C + 1e-12 * np.trace(C) / d * np.eye(d)
    sd = np.sqrt(np.diag(C))
    assert r.stats()["whiten_fallbacks"] == 0
    assert np.abs((L @ L.T - C) / np.outer(sd, sd)).max() < (20 + d) * np.finfo(float).eps * 4
    r.close()
