"""The autotuner's candidates, without a GPU: the library's own choice of reducers is one of
them, so that a tuned call is not held to reducers beside launches that do without."""
import torch

from paper_1912_05529_amd import mig, tune


def test_candidates_include_the_librarys_choice(monkeypatch):
    seen = []

    class Event:
        def __init__(self, enable_timing):
            pass

        def record(self, stream):
            pass

        def synchronize(self):
            pass

        def elapsed_time(self, other):
            return 1.0 if seen[-1]["reducers"] == 0 else 2.0

    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: None)
    monkeypatch.setattr(mig, "batch_workspace_size", lambda batch, desc, tune: 1)
    monkeypatch.setattr(mig, "migrate_batched", lambda batch, tab32, desc, tune, ws: seen.append(tune))

    class Desc:
        ntaps, nk = 35, 64

    batch = [{"data": torch.empty(4, 2), "vel": torch.empty(3, 4)}]
    best, table = tune.autotune(batch, torch.empty(1), Desc, reps=1, use_cache=False)
    assert best["reducers"] == 0
    assert {r["tune"]["reducers"] for r in table} == set(tune.REDUCERS)
