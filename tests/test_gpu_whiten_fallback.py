"""The whitening factor's fallback where a pivot beyond the first block of sixteen columns fails.

The first `healthy` coordinates are independent normals, so their pivots are as large as their
variances.  The others are the same for every survivor but the best point, about which the sums are
taken: their block has rank one, its variances are D^2 / n (D: the distance to the best point, n
survivors), the jitter 1e-12 of that, 2e-16 D^2 at n = 5000, while the sums' rounding is a few units
of 1e-16 D^2 for each pair on its own.  Of the dozens of pivots that are nothing but rounding some
are negative: the factor has to be the diagonal one, with the entries of the blocks already stored
cleared.  The sums round by at most 1e-14
of D^2, 5e-11 of the variances D^2 / n: their bar is 1e-9."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d, healthy", [(48, 20), (128, 40), (128, 100)])
def test_failing_pivot_in_a_later_block(d, healthy):
    from paper_2601_23252_amd import nss, problems as G
    m, k = 6000, 1000
    n = m - k
    prob = G.gaussian_problem(d, np.zeros(d), 0.04 * np.eye(d), "box", -10.0, 10.0, m=m, k=k)
    rng = np.random.default_rng(d + healthy)
    x = np.empty((m, d))
    x[:, :healthy] = rng.normal(size=(m, healthy)) / np.sqrt(n)
    x[:, healthy:] = rng.uniform(0.5, 1.5, d - healthy)
    x[-1, healthy:] = 0.0
    L = -np.arange(m, 0, -1.0)
    r = nss.NSRun(prob, m=m, k=k, p=1, seed=1)
    s = r.state()
    r.set_state(x, L, s["logZ"], s["logX"], s["M"], s["iter"])
    r.step()
    Ls = r.state()["Lsig"]
    assert r.stats()["whiten_fallbacks"] == 1
    r.close()
    assert np.all(Ls[~np.eye(d, dtype=bool)] == 0.0)
    assert np.allclose(np.diag(Ls), x[k:].std(axis=0), rtol=1e-9, atol=0)
