"""What the benchmark's records call a rate: achieved bytes only where the bytes are those
that move."""
import os
import sys
import types

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)
import bench  # noqa: E402
from paper_1510_07328_amd import inputs, lbm  # noqa: E402


def test_boxes_with_several_steps_per_pass_report_an_equivalent_rate(monkeypatch):
    lat = types.SimpleNamespace(totals=lambda: [1.0], free=lambda: None)
    monkeypatch.setattr(bench, "timed_run", lambda *a, **k: (lat, 10.0, 0.0, 4096, 19, 622592))
    monkeypatch.setattr(inputs, "perturbed_field", lambda *a, **k: (None, None))
    for lattice, shape in (("d2v9", (64, 64, 1)), ("d3v19", (16, 16, 16))):
        rec = bench.extra_record(lbm, None, inputs, lattice, shape, 100, 4.0, 0.6, "box", autotune=False)
        assert "achieved_GBs" not in rec and "frac" not in rec and rec["equivalent_GBs"] > 0
    rec = bench.extra_record(lbm, None, inputs, "d2v41", (64, 64, 1), 100, 4.0, 0.6, "box", autotune=False)
    assert rec["achieved_GBs"] > 0


def test_recorded_traffic_is_that_of_the_timed_call():
    """Passes of a call of 20 steps are not those of a long call; other calls were not measured."""
    for scheme in ("aa", "push"):
        short, long = bench.measured_traffic(scheme, 20), bench.measured_traffic(scheme, 200)
        assert short > 1.1 * long and bench.measured_traffic(scheme, 10000) == long
        assert bench.measured_traffic(scheme, 30) is None and bench.measured_traffic(scheme, 201) is None
    # after an odd warm-up an AA call starts and ends with a single step
    assert bench.measured_traffic("aa", 20, 5) > 1.3 * bench.measured_traffic("aa", 20, 4)
    assert bench.measured_traffic("push", 20, 5) == bench.measured_traffic("push", 20)
