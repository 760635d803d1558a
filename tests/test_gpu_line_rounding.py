"""Decisions of the line-evaluating chain kernel where a form at the candidate is far smaller than at
the chain's point: a form's rounding is relative to the larger one, and must not decide.

The states are laid out from the counter-based draws: chain j's parent is placed so that one
candidate of its first step falls on a chosen point y*, whose log L the threshold L* lies close to.
The point-evaluating kernels (NS_FLAG_SHALLOW_PLAN) find every such candidate inside the slice; the
chains must be theirs, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

M, K, SEED = 32, 8, 7
RESAMPLE, DIR, STEP = 2, 3, 4


def _parents(O):
    """Chain j's parent with survivors K..M-1 in order (the first iteration's draws)."""
    u = [O.uniform_pair(SEED, 0, RESAMPLE, j, 1, 0, 0)[0] for j in range(K)]
    return [K + min(int(v * (M - K)), M - K - 1) for v in u]


def _direction(O, j, step, d):
    z = []
    for q in range((d + 1) // 2):
        ua, ub = O.uniform_pair(SEED, 0, DIR, j, 1, step, q)
        r = np.sqrt(-2.0 * np.log(ua))
        z += [r * np.cos(2 * np.pi * ub), r * np.sin(2 * np.pi * ub)]
    return np.array(z[:d])


def _run(prob, y, moves, parents, Lstar, scale, shallow, **kw):
    """One iteration from a state where chain j's parent is y - moves[j] (the first chain of a
    shared parent counts): state after it, trace, counters."""
    from paper_2601_23252_amd import nss
    d = prob["d"]
    x = np.tile(np.asarray(y, float), (M, 1))
    for j in reversed(range(K)):
        x[parents[j]] = y - moves[j]
    logL = np.full(M, Lstar - 1.0)
    logL[K - 1] = Lstar
    logL[K:] = Lstar + 1.0 + 1e-3 * np.arange(M - K)
    R = nss.NSRun(prob, m=M, k=K, p=4, seed=SEED, trace=True, freeze_whitening=True,
                  shallow_plan=shallow, term_frac=0.0, **kw)
    R.set_state(x, logL, -np.inf, 0.0, 0.0, 0, Lsig=scale * np.eye(d))
    assert R.state()["Lstar"] == Lstar
    R.step()
    s, tr = R.state(), R.trace()
    R.close()
    return s, tr


def _same_as_points(prob, y, moves, parents, Lstar, scale, **kw):
    a, ta = _run(prob, y, moves, parents, Lstar, scale, False, **kw)
    b, tb = _run(prob, y, moves, parents, Lstar, scale, True, **kw)
    assert np.array_equal(ta, tb)
    assert np.array_equal(a["x"], b["x"])
    assert np.array_equal(a["logL"], b["logL"])
    return tb


def _slice_moves(O, d, scale, width):
    """t v of the first step's left end."""
    out = []
    for j in range(K):
        z = _direction(O, j, 0, d)
        t = -width * O.uniform_pair(SEED, 0, STEP, j, 1, 0, 0)[0]
        out.append(t * scale * z / np.linalg.norm(z))
    return out


@pytest.mark.parametrize("rw", [False, True])
def test_funnel_neck(oracle_lib, rw):
    """From the mouth (radius about 10) into the neck at v = -18: exp(18) weighs the radius'
    square, so 1e-14 of the mouth's there is 1e-6 of log L."""
    from paper_2601_23252_amd import problems as G
    O = oracle_lib
    prob = G.funnel(2, m=M, k=K, p=4)
    y = np.array([-18.0, 1e-5])
    Lstar = O.Problem(prob).loglik(y[None])[0] - 1e-8
    if rw:
        scale, kw = 8.0, dict(replacement="rw", width=1.0)
        moves = [scale * _direction(O, j, 0, 2) for j in range(K)]
    else:
        scale, kw = 30.0, dict(width=1.0)
        moves = _slice_moves(O, 2, scale, 1.0)
    parents = _parents(O)
    tr = _same_as_points(prob, y, moves, parents, Lstar, scale, **kw)
    first = [parents.index(p) for p in set(parents)]
    inside = [np.all(np.abs(y - moves[j]) <= 20.0) for j in first]
    hits = sum((tr[j, 0, 3] if rw else tr[j, 0, 0]) > 0 for j in first)
    assert hits >= max(2, sum(inside) // 2)


@pytest.mark.parametrize("rw", [False, True])
def test_narrow_far_component(oracle_lib, rw):
    """A component of width 1e-9 three away: its form is 1e18 at the chain's point and 0.5 at the
    candidate, where L* lies 10 below log L."""
    from paper_2601_23252_amd import problems as G
    O = oracle_lib
    prob = dict(G.mixture_problem(1, 2, 2, m=M, k=K, p=4), mu=np.array([[0.0, 0.0], [3.0, 1.0]]),
                cov=np.array([np.eye(2), 1e-18 * np.eye(2)]))
    y = np.array([3.0 + 5e-10, 1.0 - 5e-10])
    Lstar = O.Problem(prob).loglik(y[None])[0] - 10.0
    scale = 4.0
    if rw:
        kw = dict(replacement="rw", width=1.0)
        moves = [scale * _direction(O, j, 0, 2) for j in range(K)]
    else:
        kw = dict(width=1.0)
        moves = _slice_moves(O, 2, scale, 1.0)
    tr = _same_as_points(prob, y, moves, _parents(O), Lstar, scale, **kw)
    assert np.sum((tr[:, 0, 3] if rw else tr[:, 0, 0]) > 0) >= 3


def test_a_point_on_the_contour_is_not_kept(oracle_lib):
    """L* equal to the last proposal's own log L, to the last bit: the proposal is not above it,
    and the chain keeps its parent, whatever a form's last bits say."""
    from paper_2601_23252_amd import problems as G
    O = oracle_lib
    d = 5
    prob = G.gaussian_problem(d, np.zeros(d), 0.09 * np.eye(d), "box", -20.0, 20.0, m=M, k=K, p=4)
    kw = dict(replacement="rw", width=1.0)
    scale = 1.5
    y = np.full(d, 0.01)
    moves = [scale * _direction(O, j, 3, d) for j in range(K)]   # the last step's proposal
    parents = _parents(O)
    below = O.Problem(prob).loglik(y[None])[0] - 1e-3
    s, tr = _run(prob, y, moves, parents, below, scale, True, **kw)
    chains = [j for j in range(K) if parents.index(parents[j]) == j and tr[j, 3, 3] == 1]
    assert len(chains) >= 5
    for j in chains:
        Lstar = s["logL"][j]   # chain j's slot: the deleted points are 0..K-1, L* the last
        a, _ = _run(prob, y, moves, parents, Lstar, scale, False, **kw)
        b, _ = _run(prob, y, moves, parents, Lstar, scale, True, **kw)
        assert np.all(a["logL"] > Lstar)
        assert np.array_equal(a["x"], b["x"])
        assert np.array_equal(a["logL"], b["logL"])


@pytest.mark.parametrize("edge, scale", [(1e39, 1e38), (1e35, 1e34), (1e-33, 1e-34), (1.0, 1e39),
                                         (1.0, 1e33), (1e-3, 1e-36)])
def test_boxes_beyond_single_precision(edge, scale):
    """Box edges, directions and their quotients outside FP32's range: the same proposals are in
    the box as for the point-evaluating kernels, which test every coordinate in FP64.  (The
    likelihood's width is the box's; 400 shrinks bring t from 1 to below 1e-40.)"""
    from paper_2601_23252_amd import nss, problems as G
    d = 3
    prob = G.gaussian_problem(d, np.zeros(d), (0.3 * edge) ** 2 * np.eye(d), "box", -edge, edge,
                              m=M, k=K, p=9)
    out = []
    for shallow in (False, True):
        R = nss.NSRun(prob, m=M, k=K, p=9, seed=SEED, trace=True, freeze_whitening=True,
                      shallow_plan=shallow, shrink_cap=400, term_frac=0.0)
        s = R.state()
        R.set_state(s["x"], s["logL"], -np.inf, 0.0, 0.0, 0, Lsig=scale * np.eye(d))
        R.step()
        t = R.stats()
        out.append((R.state(), R.trace(), [t[q] for q in ("evals", "tests", "prior_rejects",
                                                          "shrink_caps")]))
        R.close()
    (a, ta, ca), (b, tb, cb) = out
    assert np.array_equal(ta, tb) and ca == cb
    assert np.array_equal(a["x"], b["x"]) and np.array_equal(a["logL"], b["logL"])
    assert np.all(np.abs(a["x"]) <= edge)
