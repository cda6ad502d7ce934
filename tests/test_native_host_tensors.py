"""Host tensors are refused by every entry point that takes device tensors, before any library call
that would launch a kernel on their addresses. The library is replaced by a proxy that lets only the
host-side calls through and the GPU queries by stubs, so nothing here can reach a GPU."""
import pytest
import torch

import synth
from paper_2408_03204_amd import (GradStep, RenderBuffers, Schedule, delay_phasor_regularise, encoder,
                                  mrstft_loss, render)
from paper_2408_03204_amd import api, load
from paper_2408_03204_amd.api import render_noalloc

HOST_CALLS = ("grafx_schedule_free", "grafx_workspace_bytes", "grafx_mrstft_workspace_bytes",
              "grafx_encoder_sizes", "grafx_last_error")
T = 4096


class HostOnly:
    def __getattr__(self, name):
        def launched(*_):
            raise AssertionError(f"{name} called with host tensors")
        return getattr(load(), name) if name in HOST_CALLS else launched


@pytest.fixture
def console(monkeypatch):
    w = synth.tiny_console(T=T)
    sched = Schedule(w.graph.node_type, w.graph.edges)
    S = torch.as_tensor(w.sources)
    P = {t: torch.as_tensor(p) for t, p in w.params.items() if p.shape[0] > 0}
    monkeypatch.setattr(api, "load", HostOnly)
    monkeypatch.setattr(encoder, "load", HostOnly)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda index: 0, raising=False)
    return sched, S, P


def with_plan(sched):
    """A plan already in place for the host device, so that a call reaches its own check."""
    sched._plans[torch.device("cpu")] = torch.empty(max(sched.plan_bytes, 256), dtype=torch.uint8)
    return sched


def rows(n):
    return torch.zeros((n, 2, T))


CALLS = {
    "plan": lambda s, S, P: s.plan("cpu"),
    "render": lambda s, S, P: render(s, S, P),
    "render with a plan": lambda s, S, P: render(with_plan(s), S, P),
    "render_noalloc": lambda s, S, P: render_noalloc(s, with_plan(s).plan("cpu"), S, P,
                                                     rows(s.num_nodes)),
    "mrstft_loss": lambda s, S, P: mrstft_loss(rows(1), rows(1)),
    "buffers": lambda s, S, P: RenderBuffers(s, T, "cpu"),
    "buffers forward": lambda s, S, P: RenderBuffers(with_plan(s), T, "cpu").forward(S, P),
    "buffers backward": lambda s, S, P: RenderBuffers(with_plan(s), T, "cpu").backward(S, P, rows(1)),
    "buffers step": lambda s, S, P: RenderBuffers(with_plan(s), T, "cpu").step(S, P, 1),
    "buffers backward_step": lambda s, S, P: RenderBuffers(with_plan(s), T, "cpu").backward_step(
        S, P, rows(1), 1),
    "buffers error_word": lambda s, S, P: RenderBuffers(with_plan(s), T, "cpu").error_word(),
    "grad step": lambda s, S, P: GradStep(with_plan(s), S, P, rows(1)).run(),
    "regularise": lambda s, S, P: delay_phasor_regularise("delay", torch.zeros((2, 220)),
                                                          torch.zeros((2, 220)), 0.1),
    "logmel": lambda s, S, P: encoder.logmel(S),
    "adam": lambda s, S, P: encoder.adam(*(torch.zeros(4) for _ in range(4)), step=1, lr=0.1),
    "encoder": lambda s, S, P: encoder.Encoder(torch.zeros(encoder.sizes(1, 8)[0]), 1, 8),
    "chain_params": lambda s, S, P: encoder.chain_params(torch.zeros((1, 11))),
}


@pytest.mark.parametrize("call", list(CALLS))
def test_host_tensors_are_refused(console, call):
    with pytest.raises(ValueError):
        CALLS[call](*console)


def test_backward_of_the_loss_refuses_a_host_tensor(console):
    ctx = type("Ctx", (), {"saved_tensors": (rows(1), rows(1)), "ws": torch.empty(256)})()
    with pytest.raises(ValueError):
        api._MRSTFT.backward(ctx, torch.ones(()))


@pytest.mark.parametrize("device", ["cpu", "meta"])
def test_stream_of_a_device_that_is_no_gpu(console, device):
    with pytest.raises(ValueError):
        api._stream(torch.device(device))


def test_stream_of_a_gpu(console):
    assert api._stream(torch.device("cuda")) == 0 and api._stream(torch.device("cuda:1")) == 0
