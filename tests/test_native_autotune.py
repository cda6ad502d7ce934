"""What the autotuner times: a recording stand-in for the render buffers (no GPU). The pointwise unroll
is chosen from whole passes, which launch chains of pointwise steps as one kernel; the other settings
from the steps of their node types."""
import pytest
import torch

import synth
from paper_2408_03204_amd import Schedule, autotune


class Recorder:
    def __init__(self):
        self.calls = []

    def forward(self, S, P):
        self.calls.append("forward")

    def backward(self, S, P, dY):
        self.calls.append("backward")

    def step(self, S, P, n):
        self.calls.append(("step", n))

    def backward_step(self, S, P, dY, n):
        self.calls.append(("backward_step", n))


class Event:
    def __init__(self, enable_timing):
        pass

    def record(self):
        pass

    def elapsed_time(self, other):
        return 1.0


@pytest.mark.parametrize("knob", [Schedule.TUNE_POINTWISE_UNROLL, Schedule.TUNE_EQ_ORDER])
def test_what_a_setting_is_timed_on(monkeypatch, knob):
    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(torch.cuda, "synchronize", lambda device: None)
    w = synth.tiny_console(T=64)
    sched, rb = Schedule(w.graph.node_type, w.graph.edges), Recorder()
    times = autotune.tune_knob(sched, knob, torch.as_tensor(w.sources), {}, reps=3, rb=rb)
    cands = autotune.KNOBS[knob][1]
    assert set(times) == set(cands)
    whole, single = rb.calls.count("forward"), [c for c in rb.calls if isinstance(c, tuple)]
    assert rb.calls.count("backward") == whole
    if knob == Schedule.TUNE_POINTWISE_UNROLL:
        assert whole == len(cands) * (1 + 1 + 3) and not single
    else:
        assert whole == len(cands) and {n for _, n in single} == {
            n for n in range(1, sched.num_steps + 1) if int(sched.step_type[n]) in (4,)}
