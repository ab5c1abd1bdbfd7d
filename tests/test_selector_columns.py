"""What the selector's labels and its evaluation compare runs on the same kernels (stubs in the place of
the solver: each call notes the launch option it would have run with)."""
from types import SimpleNamespace

import numpy as np
import pytest

from paper_1903_12085_amd import selector as S


class Graph:
    n, single = 100, 0

    def launch(self):
        return {"single": self.single}

    def set_launch(self, single):
        self.single = single


class Solver:
    """Every solver entry point of the binding that selector.py calls, noting name and launch option."""
    STATIC_OR, SIMPLE_OR, IN_SIMPLE, OUT_STATIC = 6, 24, 8, 4
    CHOICE_CRIT, CHOICE_DELTA, SELECTOR_PARAMS = (6, 24, 12), (4096, 16384, 65536), 5382

    def __init__(self):
        self.calls = []

    def new_dist(self, n):
        return None

    def Selector(self, w):
        return "static only"

    def __getattr__(self, name):
        def call(dg, *args, **kw):
            # solve_ex, the schedules, switched and per-phase learned solves know no other kernels
            always = name in ("solve_ex", "solve_schedule", "solve_switch", "solve_learned", "delta_step_learned") or \
                bool(kw.get("trace_cap"))
            self.calls.append((name, "phases" if always or dg.single == 2 else "resident"))
            r = SimpleNamespace(phases=100, trace={"criterion": np.array([6] * 50 + [12] * 50)})
            return (r, np.zeros((6, 12), np.float32)) if kw.get("features") else r
        return call


@pytest.fixture
def solver(monkeypatch):
    b = Solver()
    monkeypatch.setattr(S, "B", b)
    monkeypatch.setattr(S, "_timed", lambda fn, reps=2: (fn(), 1e-3)[1])
    return b


@pytest.mark.parametrize("single", [0, 1, 2])
def test_evaluation_compares_like_with_like(solver, single):
    dg = Graph()
    dg.single = single
    e = S.evaluate("weights", dg, 0)
    assert dg.single == single
    assert solver.calls[-2:] == [("solve", "resident"), ("solve_checkpoint", "resident")]  # *_default
    assert len(solver.calls) > 8 and {k for _, k in solver.calls[:-2]} == {"phases"}, solver.calls
    assert {"checkpoint_over_static", "checkpoint_over_static_default", "static_or_ms", "simple_or_ms"} <= set(e)


def test_labels_compare_like_with_like(solver):
    dg = Graph()
    m = S.measure(dg, 0)
    assert dg.single == 0 and m["schedules"] and len(m["delta_time"]) == 3
    assert {k for _, k in solver.calls} == {"phases"}, solver.calls


def test_launch_option_is_restored_after_an_error(solver, monkeypatch):
    dg = Graph()
    monkeypatch.setattr(S, "candidate_checkpoints", lambda phases: 1 / 0)
    with pytest.raises(ZeroDivisionError):
        S.measure(dg, 0)
    assert dg.single == 0
