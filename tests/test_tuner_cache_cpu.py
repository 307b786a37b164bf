"""Launch shapes cached before the passes they were timed against changed are not
handed out."""
from paper_2312_10318_amd import autotune


class _Member:
    nx, ny, storage, mask, inflow = 128, 128, "f64", None, None


def test_shapes_of_other_rules_are_ignored(tmp_path, monkeypatch):
    path = str(tmp_path / "tune.json")
    monkeypatch.setenv("TRTLBM_TUNE_CACHE", path)
    old = {"best": [8, 4, 1, 1, 0, 1, 0]}
    autotune.save_cache({"gfx950|f64|open|128|128": old, "gfx950|f64|open|batch|2|128x2": old})
    assert autotune.best_shape(128, 128, "f64") is None
    assert autotune.best_batch_shape([_Member, _Member]) is None
    new = {"best": [0, 0, -1, 0, 0, 0, 0]}
    autotune.save_cache({autotune.key(128, 128, "f64", False): new,
                         autotune.batch_key([(128, 128)] * 2, "f64", False): new})
    assert autotune.best_shape(128, 128, "f64") == autotune.AUTOMATIC
    assert autotune.best_batch_shape([_Member, _Member]) == autotune.AUTOMATIC
