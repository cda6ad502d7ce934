"""Dynamics at the ends of their parameters' and signals' ranges, against values known in closed form."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import say
from paper_2408_03204_amd import RenderBuffers, Schedule

pytestmark = pytest.mark.gpu


def run(kind, u, p, dY):
    """One node of `kind` on the source u [2, T] with the parameter row p: Y, dS, dP."""
    b = synth.GraphBuilder()
    i, n, o = b.add(synth.IN), b.add(kind), b.add(synth.OUT)
    b.connect(i, n)
    b.connect(n, o)
    g = b.build()
    sched = Schedule(g.node_type, g.edges)
    S = torch.as_tensor(u[None]).cuda()
    P = {kind: torch.tensor([p], dtype=torch.float32).cuda()}
    rb = RenderBuffers(sched, u.shape[1])
    dS, dP = torch.empty_like(S), {kind: torch.empty_like(P[kind])}
    rb.forward(S, P)
    rb.backward(S, P, torch.as_tensor(dY[None]).cuda(), dP, dS)
    torch.cuda.synchronize()
    return rb.Y[0].cpu().numpy(), dS[0].cpu().numpy(), dP[kind][0].cpu().numpy()


def signal(T, low, high, seed):
    """Equal channels whose samples are `low` or `high` in size."""
    rng = np.random.default_rng(seed)
    m = np.where(rng.random(T) < 0.5, low, high) * rng.choice([-1.0, 1.0], T)
    return np.stack([m, m]).astype(np.float32), np.abs(m) == high


@pytest.mark.parametrize("knee", [0.0, 0.5])
def test_noise_gate_of_infinite_ratio(knee):
    """alpha = 0: the envelope is the sample's own energy. Above the knee the gate passes the sample,
    below it the gain is 0; the gradients of a signal that lies above it are those of a wire."""
    T = 7001
    say(f"[gate, infinite ratio] knee {knee}")
    u, up = signal(T, 1e-3, 0.5, 3)  # energies 4e-6 and 1 around a threshold of -4 (0.018)
    dY = np.random.default_rng(4).standard_normal((2, T)).astype(np.float32)
    Y, _, _ = run(synth.GATE, u, [0.0, -4.0, knee, np.inf], dY)
    assert np.array_equal(Y, np.where(up, u, 0.0).astype(np.float32))
    v, _ = signal(T, 0.4, 0.5, 5)
    Y, dS, dP = run(synth.GATE, v, [0.0, -4.0, knee, np.inf], dY)
    assert np.array_equal(Y, v) and np.array_equal(dS, dY) and np.all(dP == 0.0)


@pytest.mark.parametrize("kind,alphas", [(synth.COMP, [0.0]), (synth.COMP_AR, [0.0, 0.0])])
def test_compressor_whose_ratio_has_no_finite_inverse(kind, alphas):
    """R = 1e-39 (1 / R is beyond float's range): below the knee the compressor is a wire."""
    T = 5003
    v, _ = signal(T, 1e-3, 2e-3, 6)
    dY = np.random.default_rng(7).standard_normal((2, T)).astype(np.float32)
    Y, dS, dP = run(kind, v, alphas + [-4.0, 0.5, 1e-39], dY)
    assert np.array_equal(Y, v) and np.array_equal(dS, dY) and np.all(dP == 0.0)


@pytest.mark.parametrize("kind,alphas,p", [(synth.COMP, [0.0], -0.5), (synth.COMP_AR, [0.0, 0.0], -0.5),
                                           (synth.GATE, [0.0], 1.0)])
@pytest.mark.parametrize("size", [2e18, 4e18, 9e18])
def test_adjoint_of_an_envelope_near_the_largest_float(kind, alphas, p, size):
    """alpha = 0 and a hard knee, every sample on the curve's slope: gamma = (g / e^T)^p with the
    envelope g = (u_l + u_r)^2 of 1e37 to 3e38, so ubar_c = gamma ybar_c + 2 (u_l + u_r) rho p / g,
    rho = sum_c ybar_c y_c. Tolerance: the gradients' 1e-3 of the largest entry, less the part that
    does not pass the envelope."""
    T, thr = 3100, (89.0 if kind == synth.GATE else 80.0)
    rng = np.random.default_rng(8)
    u = (rng.choice([-1.0, 1.0], (1, T)) * rng.uniform(0.8, 1.0, (2, T)) * size).astype(np.float32)
    dY = rng.standard_normal((2, T)).astype(np.float32)
    _, dS, _ = run(kind, u, alphas + [thr, 0.0, 2.0], dY)
    u64, m = u.astype(np.float64), u.astype(np.float64).sum(axis=0)
    g = m * m
    gain = np.exp(p * (np.log(g) - thr))
    through = 2.0 * m * (dY * gain * u64).sum(axis=0) * p / g
    ref = gain * dY + through
    say(f"[envelope near the largest float] kind {kind} size {size:g}: "
        f"{np.abs(dS - ref).max() / np.abs(through).max():.2e}")
    assert np.abs(dS - ref).max() <= 1e-3 * np.abs(through).max()
