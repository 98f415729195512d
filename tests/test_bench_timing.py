"""What bench.py times: the warm-up runs the form of a step that the timed region runs, and the force time that it
reports is that of the timed steps alone."""
import importlib.util
import os

import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


class FakeSim:
    """A handle in graph mode as far as the timed region sees it: the first step of a form captures it."""

    def __init__(self):
        self.captured, self.timing, self.log, self.launches, self.total = set(), False, [], 0, 0

    def set_graph_mode(self, on):
        assert on

    def enable_kernel_timing(self, on=True):
        self.timing, self.launches = on, 0

    def step(self, n):
        form = "timed" if self.timing else "whole"
        self.log.append((n, form, form not in self.captured))
        if n:
            self.captured.add(form)
        self.total += n
        self.launches += n if self.timing else 0

    def kernel_time(self):
        return 2.0 * self.launches, self.launches

    def state(self):
        return None, None, self.total, {"steps": self.total}

    def close(self):
        pass


def test_no_capture_in_the_timed_region(monkeypatch):
    spec = importlib.util.spec_from_file_location("bench_under_test", os.path.join(ROOT, "bench.py"))
    bench = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(bench)
    from paper_1703_02484_amd import binding

    sim = FakeSim()
    monkeypatch.setattr(binding.Sim, "from_workload", classmethod(lambda cls, w, **over: sim))
    monkeypatch.setattr(torch.cuda, "synchronize", lambda *a: None)
    elapsed, force_s, counters = bench._short_range_once(object(), 7, 5, "delaunay")
    assert [n for n, _, _ in sim.log] == [5, 7]      # the warm-up as asked for, then the steps as asked for
    assert not sim.log[-1][2]                        # nothing captured while the clock runs
    assert sim.launches == 7 and abs(force_s - 2e-3) < 1e-12 and counters == {"steps": 7} and elapsed >= 0.0
