"""What the tuner pins is what it timed: the library's own tiling is a candidate
of its own beside every fixed one, and a plan for which it won keeps it.  The
plan and the timer are stubs (no GPU)."""

import json
from types import SimpleNamespace

import pytest

pytest.importorskip("torch")
tuner = pytest.importorskip("paper_1910_01972_amd.tuner")
ols = pytest.importorskip("paper_1910_01972_amd.ols")


class Plan:
    """Reports 2 x 2 for the library's choice, which runs something else."""

    def __init__(self, h, N=0):
        self.N, self.fixed = N, None

    def set_tiling(self, nf, wpc):
        self.fixed = (nf, wpc or 2) if nf else None

    def tiling(self):
        nf, wpc = self.fixed or (2, 2)
        return {"filters_per_unit": nf, "workgroups_per_cu": wpc, "max_workgroups_per_cu": 2}

    def call(self, Ns, y=None):
        return {"filters_per_unit": 1, "block": 128, "grid": 1024, "hop": self.N // 2}

    def close(self):
        pass


@pytest.fixture
def stub(monkeypatch, tmp_path):
    """tune() over a table of times per tiling (None: the library's), and a cache file."""
    times = {}
    monkeypatch.setattr(ols, "OLSPlan", Plan)
    monkeypatch.setattr(tuner, "torch", SimpleNamespace(empty=lambda *a, **k: None, complex64=None))
    monkeypatch.setattr(tuner, "_time_forward", lambda plan, *a, **k: times[plan.fixed])
    monkeypatch.setattr(tuner, "_arch", lambda: "gfx950")
    data = (SimpleNamespace(shape=(1 << 20,)), None)
    return times, dict(data=data, candidates=(2048,)), str(tmp_path / "c.json")


@pytest.mark.parametrize("winner", [None, (1, 2), (2, 1), (2, 2)])
def test_choice_was_timed_as_pinned(stub, winner):
    times, kw, path = stub
    times.update({None: 1.0, (1, 1): 1.3, (1, 2): 1.1, (2, 1): 1.4, (2, 2): 1.2})
    times[winner] = 0.5
    r = tuner.tune(64, 32, **kw)
    assert r["tiling_ms"] == {"auto": times[None], "1x1": times[1, 1], "1x2": times[1, 2], "2x1": times[2, 1],
                              "2x2": times[2, 2]}
    assert r["automatic"] is (winner is None)
    cfg = tuner.TuneCache(path).config(64, 32, **kw)
    assert json.load(open(path)) == {"gfx950|M=64|K=32|max=8192": cfg}
    times.clear()  # from here on the file alone
    plan = tuner.TuneCache(path).plan(SimpleNamespace(shape=(32, 64)))
    assert plan.N == 2048 and plan.fixed == winner


def test_entries_of_uncertain_timing_are_measured_again(stub):
    times, kw, path = stub
    times.update({None: 1.0, (1, 1): 1.3, (1, 2): 1.1, (2, 1): 1.4, (2, 2): 1.2})
    old = {"N": 2048, "filters_per_unit": 2, "workgroups_per_cu": 2}
    with open(path, "w") as f:
        json.dump({"gfx950|M=64|K=32|max=8192": old,
                   "gfx950|M=64|K=8|max=8192": dict(old, N=1024),
                   "gfx950|M=64|K=4|max=8192": dict(old, filters_per_unit=1)}, f)
    c = tuner.TuneCache(path)
    assert c.config(64, 32, **kw)["automatic"] is True
    times.clear()  # the other two stand
    assert c.config(64, 8, **kw)["N"] == 1024 and c.config(64, 4, **kw)["filters_per_unit"] == 1
