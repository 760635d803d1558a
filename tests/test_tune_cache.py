"""The tuner's cache file and the kernel an entry was tuned for (host only)."""
import json

import pytest

ENTRY = dict(D=64, lik=1, mode=3, upw=8, rw=0, chains=1000, planned=1, C=4, plan=16)
FP64 = dict(D=32, lik=2, mode=0, upw=1, rw=0, chains=77, planned=0, C=2, plan=0)


def _write(path, *entries):
    path.write_text('{"nss_tune": 2, "entries": [' + ",".join("\n  " + json.dumps(e) for e in entries)
                    + "\n]}\n")
    return path


@pytest.fixture
def N():
    from paper_2601_23252_amd import nss
    assert nss.ns_tune_clear()[0] == nss.NS_OK
    yield nss
    nss.ns_tune_clear()


def test_entries_of_different_kernels_stay_apart(N, tmp_path):
    entries = [ENTRY, dict(ENTRY, kernel=1), FP64, dict(FP64, kernel=0), dict(FP64, C=3, kernel=1),
               dict(FP64, C=1, kernel=3)]
    assert N.ns_tune_load(_write(tmp_path / "a.json", *entries)) == (N.NS_OK, 6)
    assert N.ns_tune_save(tmp_path / "b.json") == (N.NS_OK, 6)
    saved = json.loads((tmp_path / "b.json").read_text())["entries"]
    assert all(e in saved for e in entries)


@pytest.mark.parametrize("bad", [dict(ENTRY, kernel=2), dict(ENTRY, kernel=-1), dict(FP64, kernel=4),
                                 dict(FP64, kernel=0.5), dict(FP64, kernel=1, more=1)])
def test_unknown_kernels_are_refused(N, tmp_path, bad):
    assert N.ns_tune_load(_write(tmp_path / "bad.json", FP64, bad))[0] == N.NS_EINVAL
    assert N.ns_tune_save(tmp_path / "b.json") == (N.NS_OK, 0)
