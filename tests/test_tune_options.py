"""Host check (no GPU): the autotuner's options for choices that no longer exist are still
accepted, and so are their entries in a table."""
import json

import pytest

from paper_1904_05575_amd import _lib as L
from paper_1904_05575_amd import tune


def test_batch_sweep_only_keeps_the_table(tmp_path, monkeypatch, capsys):
    out = tmp_path / "table.json"
    monkeypatch.setattr("sys.argv", ["tune", "--batch-sweep-only", "--reps", "1", "--out", str(out)])
    assert tune.main() == 0
    assert json.loads(out.read_text()) == json.load(open(tune.TABLE))
    assert json.loads(capsys.readouterr().out)["out"] == str(out)


@pytest.mark.parametrize("site,choice", [("batch_sweep", 0), ("batch_sweep", 4), ("batch_align", 1)])
def test_retired_entries_are_accepted(site, choice):
    old = L.bse_tune_get()
    try:
        entry = (L.TUNE_SITES[site], 5184, choice)
        L.bse_tune_set([entry])
        assert L.bse_tune_get() == [entry]
    finally:
        L.bse_tune_set(old)
