"""The launch-shape tuner's choices, on a tracker whose times are made up."""
import numpy as np
import pytest

from paper_1712_09416_amd import autotune as A


class FakeStream:
    pass


@pytest.fixture
def built(monkeypatch):
    """The shapes of the trackers built; a replay's time is `built.ms(shape)`."""
    class Built(list):
        ms = staticmethod(lambda shape: 1.0)

    b = Built()

    class FakeTracker:
        def __init__(self, geometry, max_events, max_clusters, **cand):
            A.default_params(max_events=max_events, max_clusters=max_clusters, **cand)
            b.append(cand)
            self.stream = FakeStream()

        def __getattr__(self, name):
            return lambda *a: None

        def get_tracks(self, slot, event):
            return np.zeros(1, np.int32), np.zeros(1, np.int32)

    class FakeEvent:
        def __init__(self, enable_timing):
            pass

        def record(self, stream):
            pass

        def elapsed_time(self, other):
            return 5.0 * b.ms(b[-1])

    monkeypatch.setattr(A, "Tracker", FakeTracker)
    monkeypatch.setattr(A.torch.cuda, "Event", FakeEvent)
    monkeypatch.setattr(A.torch.cuda, "synchronize", lambda: None)
    return b


def tune(**kw):
    return A.autotune({}, np.array([0, 10]), None, None, None, None, reps=5, **kw)


def test_knob_without_effect_is_timed_once_and_never_chosen(built):
    """Candidates that differ in row_batch alone are one launch shape: one
    tracker is built for them, they share its time, and noise between them
    cannot change the choice."""
    built.ms = lambda shape: 0.9 if shape["row_batch"] == 16 else 1.0    # noise beyond the margin
    res = tune()
    shapes = [tuple(v for k, v in c.items() if k != "row_batch") for c in built]
    assert len(shapes) == len(set(shapes)) == 9 + 2 + 2
    assert res["best"]["row_batch"] == 8
    assert len(res["ms"]) == 9 + 2 + 2 + 2 and res["best_ms"] == 1.0


def test_other_knobs_are_chosen_by_time(built):
    built.ms = lambda shape: 0.8 if shape["tl_block"] == 128 and shape["bin_target"] == 0.5 else 1.0 - \
        0.05 * (shape["bin_target"] == 0.5)
    best = tune()["best"]
    assert best["tl_block"] == 128 and best["bin_target"] == 0.5 and best["win_batch"] == 4


def test_invalid_value_of_the_knob_without_effect_is_refused(built):
    with pytest.raises(ValueError):
        tune(knobs={"row_batch": (8, 5)})
