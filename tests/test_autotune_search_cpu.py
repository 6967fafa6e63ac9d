"""The autotuner searches only knobs that reach a launch, on the CPU."""
import itertools

from paper_2204_12876_amd import autotune as at

START = {"grid_move": 1024, "grid_chunk": 4096, "grid_tile": 65536, "grid_setup": 4096,
         "grid_march": 8192, "grid_cells": 4096, "seg": 16, "graph": 1}


def test_default_search_leaves_knobs_without_effect_alone(monkeypatch):
    # every later candidate looks clearly faster, as noise now and then does
    calls, clock = [], itertools.count()

    def time_tuning(run_batch, tuning, reps=8, repeats=3, device=None):
        calls.append(dict(tuning))
        return 0.9 ** next(clock)

    monkeypatch.setattr(at, "time_tuning", time_tuning)
    best, _, _ = at.autotune(None, START)
    for knob in ("grid_move", "seg"):
        assert {c[knob] for c in calls} == {START[knob]}, knob
        assert best[knob] == START[knob]
    for knob in ("grid_chunk", "grid_tile", "grid_setup", "grid_march", "grid_cells"):
        assert len({c[knob] for c in calls}) > 1, knob
