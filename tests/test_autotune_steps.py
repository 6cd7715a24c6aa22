"""What the field autotuner times: single steps, the only ones whose workgroup size it sets."""
import types

import torch

from paper_1510_07328_amd import autotune as A
from paper_1510_07328_amd import lbm


def test_the_field_timer_takes_calls_of_one_step(monkeypatch):
    calls = []

    class Event:
        def __init__(self, enable_timing):
            pass

        def record(self, stream):
            calls.append("event")

        def elapsed_time(self, other):
            return 0.5

    def create(cfg, n0, u0):
        calls.append(cfg.block)
        return types.SimpleNamespace(step=lambda n: calls.append(("step", n)), stream=None, free=lambda: None)

    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda: None)
    monkeypatch.setattr(lbm.Lattice, "create", create)
    cfg = lbm.make_config("d2v9", shape=(2048, 2048, 1))
    assert A.time_field_block(cfg, None, None, 512, steps=20) == 25.0
    assert calls[0] == 512 and cfg.block == 0
    first, last = (i for i, c in enumerate(calls) if c == "event")
    assert calls[first + 1:last] == [("step", 1)] * 20
    assert {c for c in calls[1:] if c != "event"} == {("step", 1)}
