"""The tuner times the plans that its table decides: solid-harmonic ones."""
import pytest

from paper_2307_03452_amd import autotune, eri4

pytestmark = pytest.mark.gpu


def test_tuner_times_solid_plans(monkeypatch):
    made = []
    solid = eri4.SolidPlan

    class Spy(solid):
        def __init__(self, *a, tune_file=None, **k):
            made.append(tune_file)
            super().__init__(*a, tune_file=tune_file, **k)

    monkeypatch.setattr(eri4, "SolidPlan", Spy)
    entries, timings = autotune.tune([(4, 4, 4, 5)], reps=1, log=lambda m: None, buckets=[(1, 1, 1)])
    assert made[0] is None and len(made) > 4 and all(made[1:])
    t = timings[0]
    assert set(t["candidates_ms"]) == {"4x16/box", "2x16/box", "1x16/box", "2x16/slab", "1x16/slab"}
    assert t["best_ms"] == min(t["candidates_ms"].values())
    e = entries[0]
    assert t["candidates_ms"]["%dx16/%s" % (e["rows16"], e["layout"])] == t["best_ms"]
