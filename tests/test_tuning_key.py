"""The autotuner cache's key (CPU): an entry serves only problems for which the built-in rule that
it was measured against makes the same choice."""
import types

import pytest

import paper_1402_4089_amd as hmc
from paper_1402_4089_amd import tuning


def _prob(n=20000, p=1000, K=10, xfmt=hmc.HMC_X_F32, link=0, pin=1):
    return types.SimpleNamespace(n=n, p=p, K=K, xfmt=xfmt, link=link,
                                 desc=hmc.hmc_problem(n=n, p=p, K=K, xfmt=xfmt, link=link, pin_last_class=pin))


@pytest.mark.parametrize("a,b", [
    (dict(), dict(K=2)),                                        # ten classes, one free column
    (dict(K=2), dict(K=2, pin=0)),                              # one free column, two
    (dict(n=513, p=31, K=4), dict(n=900, p=32, K=4)),           # one workgroup for updates, not
    (dict(n=8192, p=100, K=2), dict(n=8000, p=100, K=2)),       # one-column pass from 8192 rows on
    (dict(n=20000, p=128, K=1, link=1, pin=0), dict(n=20000, p=120, K=1, link=1, pin=0)),
])
def test_problems_of_other_choices_do_not_share_an_entry(a, b, tmp_path, monkeypatch):
    monkeypatch.setenv(tuning.ENV, str(tmp_path / "t.json"))
    entry = {"tuning": {"path": 1, "waves": 16, "mb": 4, "grid": 250, "rows_per_slice": 0}}
    tuning._write(str(tmp_path / "t.json"), {tuning.key_of(_prob(**a)): entry})
    assert tuning.lookup(_prob(**a)) == entry["tuning"]
    assert tuning.lookup(_prob(**b)) is None


def test_an_entry_of_an_earlier_build_is_not_used(tmp_path, monkeypatch):
    monkeypatch.setenv(tuning.ENV, str(tmp_path / "t.json"))
    old = "xfmt=1:nb=1:nblk=63:n<=32768:link=0"                 # the key before it held a version
    tuning._write(str(tmp_path / "t.json"), {old: {"tuning": {"path": 1, "waves": 16, "mb": 4, "grid": 250,
                                                             "rows_per_slice": 0}}})
    assert tuning.lookup(_prob(K=2)) is None and tuning.lookup(_prob()) is None
