"""The tuner times launches that take the configuration it tunes: FP64 and FP32
step one at a time (longer runs go in pairs, which take none of it)."""
import pytest

from paper_1810_09299_amd import autotune


class _Handle:
    stream = None

    def __init__(self, precision):
        self.precision, self.runs = precision, []

    def step(self, n):
        self.runs.append(n)

    def record(self, stream):
        self.runs.append("event")

    def elapsed_time(self, other):
        return 1.0

    set_config = set_tile = close = lambda self, *a: None


@pytest.mark.parametrize("precision,chunk", [("fp64", 1), ("fp32", 1), ("fp16", 100)])
def test_batch_tuner_times_single_steps(monkeypatch, precision, chunk):
    seen = []
    monkeypatch.setattr(autotune, "time_batch", lambda b, n, steps: seen.append((n, steps)) or len(seen))
    best, timings = autotune.tune_batch(lambda: _Handle(precision), tiles=(8, 4), persistent=(0,), schedules=(1,),
                                        bands=(16,))
    assert best == (8, 0, 1, 16) and len(timings) == 2
    assert set(seen) == {(chunk, 200)}


@pytest.mark.parametrize("precision,timed", [("fp64", [1] * 200), ("fp32", [1] * 200), ("fp16", [200])])
def test_case_tuner_times_single_steps(monkeypatch, precision, timed):
    import torch
    c = _Handle(precision)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    monkeypatch.setattr(autotune, "_events", lambda: (c, c))
    assert autotune.tune_case(lambda: c, tiles=(8,)) == 8
    first = c.runs.index("event")
    assert c.runs[first + 1:] == timed + ["event"]
