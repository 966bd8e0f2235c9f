"""The schedule tuner's choice, and which kernels the bench's counter
summaries speak for (CPU only: timings are given)."""
import types

import pytest

from paper_2508_06768_amd import autotune as A


class FakeStep:
    def __init__(self):
        fan = types.SimpleNamespace(n_rays=256, n_samples=1024)
        self.geom = types.SimpleNamespace(fans=[fan])
        self.schedule = {"fwd_chunk": 0, "bwd_chunk": 4, "xcd_group": 16, "scatter_rays": 0, "span_samples": 4096}

    def get_schedule(self):
        return dict(self.schedule)

    def set_schedule(self, **s):
        self.schedule = dict(s)


@pytest.mark.parametrize("gain,taken", [(0.006, False), (0.0099, False), (0.011, True), (0.1, True)])
def test_tuner_ignores_noise(monkeypatch, gain, taken):
    step = FakeStep()
    monkeypatch.setattr(A, "shape_key", lambda geom: "key")
    monkeypatch.setattr(A, "_time", lambda fn, reps: 0.43 * (1.0 - gain * (step.schedule["bwd_chunk"] == 8)))
    out = A.autotune(step, lambda: None, use_cache=False)
    assert (out["schedule"]["bwd_chunk"] == 8) == taken
    assert step.schedule == out["schedule"]
    assert {k: v for k, v in out["schedule"].items() if k != "bwd_chunk"} == \
        {"fwd_chunk": 0, "xcd_group": 16, "scatter_rays": 0, "span_samples": 4096}


def test_tuner_looks_again(monkeypatch):
    """A schedule first timed on slow clocks is not given up for an equal."""
    step = FakeStep()
    monkeypatch.setattr(A, "shape_key", lambda geom: "key")
    calls = []
    monkeypatch.setattr(A, "_time", lambda fn, reps: calls.append(1) or (0.43 if len(calls) > 2 else 0.45))
    out = A.autotune(step, lambda: None, use_cache=False)
    assert out["schedule"] == FakeStep().get_schedule() and out["ms"] == 0.43


def test_bench_counters_speak_for_their_kernels():
    import bench
    s = FakeStep().get_schedule()
    assert all(bench.profiled_schedule(k, s) for k in ("forward", "adjoint", "scatter"))
    assert not bench.profiled_schedule("adjoint", dict(s, bwd_chunk=8))
    assert not bench.profiled_schedule("forward", dict(s, fwd_chunk=4))
    assert not bench.profiled_schedule("scatter", dict(s, scatter_rays=8))
