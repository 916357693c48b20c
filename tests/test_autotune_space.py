"""The shipped tuning cache is one that the shipped autotuner can write: every
class in it is one that a default run tunes, every setting one of the
candidates, and a run keeps the classes that it does not tune."""
import pytest

import paper_2309_03912_amd as hdc
from paper_2309_03912_amd import autotune

CACHE = autotune.read_cache(hdc.TUNING_CACHE)


def reachable(op):
    """The settings that a run's stages can end at, as sets per stage of field groups."""
    cands = autotune.candidates(op)
    return cands if isinstance(cands, tuple) else (cands,)


def test_every_class_is_tuned():
    tuned = {(op, dt, acc, hdc.tuning_bucket(n)) for op, dt, acc, n in autotune.default_classes()}
    assert sorted(set(CACHE) - tuned) == []


@pytest.mark.parametrize("key", sorted(CACHE), ids=lambda k: "_".join(map(str, k)))
def test_every_setting_is_a_candidate(key):
    op, line = key[0], CACHE[key]
    for stage in reachable(op):
        fields = set(stage[0])
        if op == hdc.OP_SEGMENTED_REDUCE and line["passes"] == 1:
            fields -= {"small_seg", "seg_per_wave"}  # of the planned schedule
        assert any(all(c[f] == line[f] for f in fields) for c in stage), (key, line)


def test_a_run_keeps_the_other_classes(tmp_path, monkeypatch):
    out = tmp_path / "cache.txt"
    autotune.write_cache(out, CACHE)
    monkeypatch.setattr(autotune, "default_classes", lambda quick, log2n: [])
    autotune.main(["--out", str(out)])
    assert autotune.read_cache(out) == CACHE
    autotune.main(["--out", str(out), "--fresh"])
    assert autotune.read_cache(out) == {}
