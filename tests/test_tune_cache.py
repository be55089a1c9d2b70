"""The tuner's cache (no GPU needed): an entry holds for the library that it was
timed with; one of another library, or from before entries named it, is not
reapplied."""
import json

import pytest

tune = pytest.importorskip("paper_1010_4124_amd.tune")


@pytest.fixture(autouse=True)
def _file(tmp_path, monkeypatch):
    monkeypatch.setenv("LBM_TUNE_CACHE", str(tmp_path / "tune.json"))


def test_entry_of_this_library_is_found():
    tune._keep("k", {"variant": 3, "ms": {"3": 0.5}})
    hit = tune._cached("k", 4)
    assert hit["variant"] == 3 and hit["ms"] == {"3": 0.5} and hit["cached"]
    assert tune._cached("k", 3) is None and tune._cached("other", 4) is None


@pytest.mark.parametrize("rec", [{"variant": 3, "ms": {}}, {"variant": 3, "library": "0" * 16}, 3])
def test_other_entries_are_not(rec):
    with open(tune.cache_path(), "w") as fh:
        json.dump({"k": rec}, fh)
    assert tune._cached("k", 27) is None
    tune._keep("k", {"variant": 1})
    assert tune._cached("k", 27)["variant"] == 1
    assert list(json.load(open(tune.cache_path()))) == ["k"]


def test_signature_changes_with_the_variants(monkeypatch):
    sig = tune.library_signature()
    tune.library_signature.cache_clear()
    monkeypatch.setattr(tune.lbm, "lbm_step_variant_count", lambda: 1)
    assert tune.library_signature() != sig
    tune.library_signature.cache_clear()
