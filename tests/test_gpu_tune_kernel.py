"""A tuned launch shape holds for the kernel it was timed on."""
import json

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def N():
    from paper_2601_23252_amd import nss
    nss.load()
    assert nss.ns_tune_clear()[0] == nss.NS_OK
    yield nss
    nss.ns_tune_clear()


def test_an_entry_tuned_on_points_does_not_hold_line_chains(N, tmp_path):
    """Two components at d = 64 in BF16x3 (k = 50): a file that names no kernel and says 8 tests was
    tuned on the point-evaluating kernels; the chains are tuned anew, a chosen shape is saved with
    its kernel, and a context that loads it back times nothing."""
    from paper_2601_23252_amd import problems as G
    prob = G.mixture_problem(3, 64, 2, m=120, k=50, p=15)
    kw = dict(precision="bf16x3", autotune=True)
    probe = N.NSRun(prob, **kw)
    probe.step()
    probe.close()
    path = tmp_path / "t.json"
    N.ns_tune_save(path)
    (entry,) = json.loads(path.read_text())["entries"]
    assert entry["kernel"] == 1
    N.ns_tune_clear()
    stale = {k: v for k, v in entry.items() if k != "kernel"}
    stale.update(C=1, plan=8)
    (tmp_path / "stale.json").write_text('{"nss_tune": 2, "entries": [\n  ' + json.dumps(stale) + "\n]}\n")
    assert N.ns_tune_load(tmp_path / "stale.json")[0] == N.NS_OK
    a = N.NSRun(prob, **kw)
    assert a.launch_shape()[1] == 16
    a.step()
    assert a.stats()["tune_launches"] > 0
    a.close()
    N.ns_tune_clear()
    assert N.ns_tune_load(path)[0] == N.NS_OK
    b = N.NSRun(prob, **kw)
    assert b.launch_shape() == (entry["C"], entry["plan"] or 4)
    b.step()
    assert b.stats()["tune_launches"] == 0
    b.close()


def test_point_and_line_chains_are_tuned_apart(N):
    """The same FP64 shape with and without NS_FLAG_SHALLOW_PLAN, and in the tempered loop."""
    from paper_2601_23252_amd import problems as G
    prob = G.config1()
    for kw in (dict(), dict(shallow_plan=True), dict(outer="smc", m=50, p=20),
               dict(outer="smc", m=50, p=20, shallow_plan=True)):
        for launches in (8, 0):
            r = N.NSRun(prob, autotune=True, **kw)
            r.step()
            assert r.stats()["tune_launches"] == launches, (kw, launches)
            r.close()
