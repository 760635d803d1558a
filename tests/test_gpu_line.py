"""The chains evaluated along each step's line (k_hrss_line) against the point-evaluating kernels
(NS_FLAG_SHALLOW_PLAN), through the C ABI, at the edges of its forms: component counts around
the lanes' shares (4, 8, 16 components), dimensions around the padded ones, chains around a
block of fifteen steps, step-out caps around a pass of eight tests and shrink caps around the
buffered six and a pass of sixteen proposals, both priors, the funnel, and tempered slices.

Both take every decision on the same point x + t v; the log-likelihoods they compare differ by
FP64 rounding, about 1e-13 of the forms' values, against spreads of order one and more, so over
the 1e4 to 1e6 tests of a case a decision differs with probability below 1e-6: the trajectories
are required to be identical, bit for bit.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def N():
    from paper_2601_23252_amd import nss
    nss.load()
    return nss


def _same(N, prob, iters=4, **kw):
    a = N.NSRun(prob, seed=11, trace=True, **kw)
    b = N.NSRun(prob, seed=11, trace=True, shallow_plan=True, **kw)
    for it in range(iters):
        da, db = a.step(), b.step()
        assert da == db
        sa, sb = a.state(), b.state()
        assert np.array_equal(a.trace(), b.trace()), it
        assert np.array_equal(sa["perm"], sb["perm"]), it
        assert np.array_equal(sa["x"], sb["x"]), it
        assert np.array_equal(sa["logL"], sb["logL"]), it
        ta, tb = a.stats(), b.stats()
        for key in ("evals", "tests", "prior_rejects", "stepout_caps", "shrink_caps",
                    "nonfinite", "band_violations"):
            assert ta[key] == tb[key], (it, key, ta[key], tb[key])
        if da:
            break
    a.close()
    b.close()


@pytest.mark.parametrize("K", [1, 4, 5, 8, 9, 16])
def test_component_counts(N, K):
    from paper_2601_23252_amd import problems as G
    _same(N, G.mixture_problem(40 + K, 20, K, m=150, k=61), p=31)


@pytest.mark.parametrize("d", [1, 2, 17, 32, 33, 64, 65, 128])
@pytest.mark.parametrize("prior", ["box", "gauss"])
def test_dimensions_and_priors(N, d, prior):
    from paper_2601_23252_amd import problems as G
    if prior == "gauss" and d > 1:
        prob = G.config2(7, d=d, m=90, k=33)
    else:
        prob = G.gaussian_problem(d, np.full(d, 0.1), 0.04 * np.eye(d), "box", -1.0, 1.0, m=90,
                                  k=33)
    _same(N, prob, p=17)


@pytest.mark.parametrize("p", [1, 3, 4, 14, 15, 16, 30])
def test_chain_lengths(N, p):
    from paper_2601_23252_amd import problems as G
    _same(N, G.mixture_problem(3, 40, 3, m=120, k=50), p=p)


@pytest.mark.parametrize("caps", [(0, 5), (1, 1), (7, 6), (8, 7), (9, 22), (10, 0), (17, 23)])
def test_caps(N, caps):
    """A narrow width, so that ends expand past one pass of eight tests, and a wide one."""
    from paper_2601_23252_amd import problems as G
    prob = G.mixture_problem(5, 12, 2, m=100, k=40)
    for width in (0.05, 60.0):
        _same(N, prob, p=18, width=width, stepout_cap=caps[0], shrink_cap=caps[1], iters=2)


@pytest.mark.parametrize("d", [2, 33, 100, 129, 320])
def test_funnel(N, d):
    from paper_2601_23252_amd import problems as G
    _same(N, G.funnel(d, m=100, k=41, p=20))


@pytest.mark.parametrize("d", [1, 2, 7, 8, 9, 64, 100, 129, 320])
@pytest.mark.parametrize("alpha", [0.0, 0.5, 1.0])
def test_rastrigin(N, d, alpha):
    from paper_2601_23252_amd import problems as G
    _same(N, G.rastrigin_gauss(d, alpha, m=100, k=41, p=20))


@pytest.mark.parametrize("p", [4, 15, 37])
@pytest.mark.parametrize("name", ["box2", "gauss17", "mix5_d33", "mix9_d20", "illcond50",
                                  "funnel9", "funnel70", "mixed64"])
def test_random_walk(N, name, p):
    """Proposals are tested a block at a time; the box cases start on wide contours (most
    proposals outside) and, with a small scale, move often within a block."""
    from paper_2601_23252_amd import problems as G
    prob, kw = {
        "box2": lambda: (G.gaussian_problem(2, np.zeros(2), 0.04 * np.eye(2), m=90, k=33), {}),
        "gauss17": lambda: (G.config2(7, d=17, m=90, k=33), {}),
        "mix5_d33": lambda: (G.mixture_problem(5, 33, 5, m=90, k=33), dict(width=0.05)),
        "mix9_d20": lambda: (G.mixture_problem(9, 20, 9, m=90, k=33), {}),
        "illcond50": lambda: (G.illcond_gaussian(50, m=90, k=33), dict(width=0.02)),
        "funnel9": lambda: (G.funnel(9, m=90, k=33), dict(width=0.3)),
        "funnel70": lambda: (G.funnel(70, m=90, k=33), {}),
        "mixed64": lambda: (G.mixture_problem(3, 64, 2, m=90, k=33), dict(precision="bf16x3")),
    }[name]()
    _same(N, prob, p=p, replacement="rw", **kw)


@pytest.mark.parametrize("target", ["gauss", "mixture", "funnel", "rastrigin"])
def test_tempered(N, target):
    from paper_2601_23252_amd import problems as G
    prob = {"gauss": lambda: G.config2(2, d=20, m=120, k=60),
            "mixture": lambda: G.mixture_problem(6, 24, 5, m=120, k=60),
            "funnel": lambda: G.funnel(9, m=120, k=60),
            "rastrigin": lambda: G.rastrigin_gauss(6, 0.5, m=120, k=60, p=20)}[target]()
    a = N.NSRun(prob, seed=4, outer="smc", p=20)
    b = N.NSRun(prob, seed=4, outer="smc", p=20, shallow_plan=True)
    for _ in range(5):
        assert a.step() == b.step()
        sa, sb = a.state(), b.state()
        # each temperature comes from sums of exp(logL), whose last bits may differ here
        assert np.allclose(sa["x"], sb["x"], rtol=0, atol=1e-10)
        assert np.allclose(sa["logL"], sb["logL"], rtol=1e-12, atol=1e-9)
        assert a.stats()["evals"] == b.stats()["evals"]
    a.close()
    b.close()


def test_limits_take_the_general_path(N):
    """Seventeen components, a prior whose squares could overflow and a Rastrigin random walk run
    (on the point-evaluating kernels)."""
    from paper_2601_23252_amd import problems as G
    _same(N, G.mixture_problem(8, 16, 17, m=80, k=20), p=9, iters=2)
    wide = G.gaussian_problem(4, np.zeros(4), np.eye(4), "box", -1e60, 1e60, m=80, k=20)
    _same(N, wide, p=9, iters=1)
    _same(N, G.rastrigin_gauss(5, 0.5, m=80, k=20, p=9), replacement="rw", iters=2)


def test_null_chains_keep_their_parents_value(N):
    """A shrink cap of zero: every step is a null move, the points and log L of the parents
    stay, also where the caller's log L is not the library's own."""
    from paper_2601_23252_amd import problems as G
    prob = G.config1()
    out = []
    for shallow in (False, True):
        r = N.NSRun(prob, seed=2, shrink_cap=0, shallow_plan=shallow)
        s = r.state()
        r.set_state(s["x"], s["logL"] - 0.25, s["logZ"], s["logX"], s["M"], s["iter"])
        r.step()
        out.append(r.state())
        r.close()
    assert np.array_equal(out[0]["logL"], out[1]["logL"])
    assert np.array_equal(out[0]["x"], out[1]["x"])
