"""Entries of the autotuner's cache count only for the table of shapes they
were chosen from: a file without the table's size and revision in its keys
(arch|kind|type|a|b, from before 8 x 8 tiles were added and NEE shape 6
took its tile from the lattice) is not applied."""
import math

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["single", "single-nee", "batch"])
def test_entries_of_another_table_are_not_applied(kind, tmp_path, monkeypatch):
    from paper_2211_05009_amd import lbm
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("LBM_TUNE_CACHE", str(path))

    def tuned():
        if kind == "batch":
            h = lbm.Batch([64, 48], [40, 64], [200.0, 200.0], dtype="f64")
            h.set_option(lbm.LBM_OPT_GRAPH_STEPS, 100)
        else:
            h = lbm.Cavity(64, 40, re=200.0, dtype="f64",
                           wall="nee" if kind == "single-nee" else "bounce-back")
        best, ms = h.autotune(chunks=1, use_cache=True)
        assert h.get_option(lbm.LBM_OPT_STEP_VARIANT) == best
        h.close()
        return best, ms

    tuned()
    line = path.read_text()
    arch, named, *rest = line.split()[0].split("|")
    path.write_text("|".join([arch, kind, *rest]) + " 0\n")
    assert not math.isnan(tuned()[1])              # timed, not taken from the file
    # this table's own entry is applied, another size's or revision's is not
    shapes, revision = named.removeprefix(kind + "/").split(".")
    key = "|".join([arch, "{}", *rest])
    for name, applied in [(f"{kind}/{shapes}.{revision}", True),
                          (f"{kind}/{int(shapes) - 1}.{revision}", False),
                          (f"{kind}/{shapes}.{int(revision) - 1}", False)]:
        path.write_text(key.format(name) + " 2\n")
        best, ms = tuned()
        assert math.isnan(ms) == applied
        assert best == 2 or not applied
