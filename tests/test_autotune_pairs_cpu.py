"""The autotuner's cache between problems that run in pairs and problems that do not (CPU, a made-up simulation)."""
import numpy as np
import pytest


@pytest.fixture
def tuner(tmp_path, monkeypatch):
    from paper_2009_12584_amd import autotune as T

    class Sim:
        def __init__(self, mask, rhoA0, rhoB0, lanes=0, **kw):
            # "pairs" problems take two steps per launch in 10 us with one lane
            self.us = 9.0 if lanes == 2 else (5.0 if mask[0, 0] else 10.0)
            self.pair_steps = 4 if mask[0, 0] and lanes != 2 else 0

        def step(self, n):
            pass

        def close(self):
            pass

    timed = []

    def time(step, sync, steps, reps=3):
        timed.append(step.__self__.us)
        return step.__self__.us

    monkeypatch.setattr(T, "_CACHE_PATH", str(tmp_path / "tune.json"))
    monkeypatch.setattr(T, "_cache", None)
    monkeypatch.setattr(T, "Simulation", Sim)
    monkeypatch.setattr(T, "_time", time)
    T.timed = timed
    yield T
    del T.timed


def problem(pairs, n=400):
    return np.full((n, n), 1 if pairs else 0, np.uint8), None, None


def test_two_lanes_are_not_carried_over_to_a_problem_that_runs_in_pairs(tuner):
    assert tuner.launch_config_for(*problem(False))["lanes"] == 2
    n = len(tuner.timed)
    assert tuner.launch_config_for(*problem(True, 300))["lanes"] == 1  # the same bucket
    assert len(tuner.timed) == 2 * n
    for pairs, lanes in ((False, 2), (True, 1)):  # both cached now
        assert tuner.launch_config_for(*problem(pairs))["lanes"] == lanes
    assert len(tuner.timed) == 2 * n


def test_models_have_their_own_entries(tuner):
    assert tuner.key_of(400, 400, 0, "f32", 1) != tuner.key_of(400, 400, 0, "f32")
    tuner.launch_config_for(*problem(False))
    n = len(tuner.timed)
    tuner.launch_config_for(*problem(False), model=1)
    assert len(tuner.timed) == 2 * n
