"""The backward has one launch shape: tuning it times that one and keeps the knob as it is."""
import json

import pytest

from paper_2603_29227_amd import tune
from paper_2603_29227_amd.ksdf import FP32


class _Model:
    precision, dense_inverse = FP32, False

    def __init__(self, lanes):
        self.now = dict(query_sub=4, query_split=1, backward_lanes=lanes)
        self.calls = 0

    def tuning(self):
        return dict(self.now)

    def set_tuning(self, **kw):
        self.now.update(kw)

    def backward(self, *args, **kw):
        self.calls += 1


@pytest.mark.parametrize("lanes", [0, 1])
def test_tune_backward_times_one_launch(lanes, tmp_path, monkeypatch):
    times = iter([2.0, 1.0])   # the second of two equal launches seems the faster

    def timed(run, reps):
        run()
        return next(times)

    monkeypatch.setattr(tune, "_median_ms", timed)
    monkeypatch.setattr(tune, "signature", lambda model, n, kind: f"{kind}|{n}")
    model, path = _Model(lanes), str(tmp_path / "cache.json")
    out = tune.tune_backward(model, [0, 0, 0], None, {}, None, cache_path=path)
    assert model.calls == 1 and model.now["backward_lanes"] == lanes
    assert out["tuning"] == {"backward_lanes": lanes} and out["ms"] == 2.0
    assert [t["ms"] for t in out["table"]] == [2.0]
    assert json.load(open(path)) == {"backward|3": {"tuning": {"backward_lanes": lanes}, "ms": 2.0}}
