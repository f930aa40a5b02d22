"""The batch measurement times replays only: a batch is launched pass by pass on the first call on it and captured on
the second, and both lie before the timed calls (no GPU: a stand-in for the library counts its calls)."""
from types import SimpleNamespace

import torch

import bench
import workloads


class _Library:
    """Call states of herk_step_batched as the library documents them, and the time each would cost."""
    BATCH_PASSES, BATCH_PER_PROBLEM = 0, 1

    def __init__(self):
        self.mode, self.calls, self.log = 0, 0, []
        lib = self

        class State:
            def __init__(self, u, dx, dt, re, scheme, n_buf):
                self.u, self.d, self.work = u, torch.zeros(1), torch.zeros(1)
                self.c = SimpleNamespace(t=0.0, work=0)

            def step(self):
                lib.log.append("single")

        self.HerkState = State

    def vor2vel(self, w, dx):
        return w

    def max_cell_speed(self, u):
        return 1.0

    def set_batch_mode(self, mode):
        self.mode, self.calls = mode, 0

    def batch_info(self):
        return (1, 1)

    def herk_step_batched(self, states):
        self.calls += 1
        first = 1 if self.mode == self.BATCH_PER_PROBLEM else 2  # (the call that captures)
        self.log.append("replay" if self.calls > first else "capture" if self.calls == first else "launch")


def test_batch_measurement_times_replays(monkeypatch):
    lib = _Library()
    spans = []

    class Event:
        def __init__(self, enable_timing):
            pass

        def record(self, stream):
            self.at = len(lib.log)

        def elapsed_time(self, end):
            spans.append(lib.log[self.at:end.at])
            return 3.0 * (1.0 + len(spans))  # (of three calls)

    cuda = SimpleNamespace(Event=Event, synchronize=lambda: None, current_stream=lambda: None)
    fake = SimpleNamespace(device=lambda name: "cpu", from_numpy=torch.from_numpy, equal=torch.equal, cuda=cuda)
    monkeypatch.setattr(workloads, "ring_edge_vorticity", lambda n, dx, ring, quad=2: torch.zeros(3, 1, 1, 1).numpy())
    out = bench.batched_measure(lib, fake, torch.float64, reps=3, sizes=(64,))
    assert [set(s) for s in spans] == [{"single"}, {"replay"}, {"replay"}]
    assert len(spans[1]) == 3 and len(spans[2]) == 3
    assert out["ms_graph_per_problem"] == 3.0 and out["ms_graph_batched_passes"] == 4.0
