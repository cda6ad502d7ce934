"""The multitap delays keep their two channels apart, though one transform carries both: each channel's
output, input adjoint and filter gradients are within the usual tolerances (renders 1e-5, gradients
1e-3, tests/gpu_common.py) of its *own* largest entry whatever the other channel's level; samples that
depend on zeros only are exact zeros; an infinity or NaN reaches the samples that depend on it and no
others. Against the FP64 oracle, both delay types; the delays run in parallel, in series and on sums."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import GRAD_TOL, RENDER_TOL, grad_err, oracle_grads, rel_err, say
from oracle import processors as OP
from oracle import render as OR
from paper_2408_03204_amd import RenderBuffers, Schedule

pytestmark = pytest.mark.gpu

KINDS = [(synth.DELAY, 5), (synth.DELAY_LONG, 20)]


def graph(kind, T, seed, series=True):
    """Two delays on one source each, one behind the second, one on the sum of both (series), or one
    delay alone."""
    b = synth.GraphBuilder()
    ins = [b.add(synth.IN) for _ in range(2 if series else 1)]
    ds = [b.add(kind) for _ in range(4 if series else 1)]
    o = b.add(synth.OUT)
    links = ((ins[0], ds[0]), (ins[1], ds[1]), (ds[1], ds[2]), (ins[0], ds[3]), (ins[1], ds[3]),
             (ds[0], o), (ds[2], o), (ds[3], o)) if series else ((ins[0], ds[0]), (ds[0], o))
    for s, d in links:
        b.connect(s, d)
    g = b.build()
    return synth.Workload("delay_channels", g, synth.make_sources(synth.rng_for(seed, 1), len(ins), T),
                          synth.draw_params(synth.rng_for(seed, 2), g), None, T, seed)


def run(w, dY):
    """Y, dS and dP [nodes][channel][slot][22] of one render and adjoint."""
    sched = Schedule(w.graph.node_type, w.graph.edges)
    S = torch.as_tensor(w.sources).cuda()
    P = {t: torch.as_tensor(p).cuda() for t, p in w.params.items() if p.shape[0] > 0}
    rb = RenderBuffers(sched, w.T)
    dS, dP = torch.full_like(S, 7.0), {t: torch.empty_like(p) for t, p in P.items()}
    rb.forward(S, P)
    rb.backward(S, P, torch.as_tensor(dY).cuda(), dP, dS)
    torch.cuda.synchronize()
    (t, p), = dP.items()
    return rb.Y.cpu().numpy(), dS.cpu().numpy(), p.cpu().numpy().reshape(p.shape[0], 2, -1, 22)


def normal(seed, *shape):
    return np.random.default_rng(seed).standard_normal(shape).astype(np.float32)


@pytest.mark.parametrize("kind,M", KINDS)
@pytest.mark.parametrize("left,right", [(1.0, 1e-3), (1e-5, 1.0), (1.0, 1e-6), (1e-30, 1.0)])
def test_channels_of_different_levels(kind, M, left, right):
    T = 11 * 474 + 100 + M * 4410
    say(f"[delay channels] M={M} levels {left:g}, {right:g}")
    w = graph(kind, T, 61)
    level = np.asarray([left, right], np.float32)[:, None]
    w.sources *= level
    dY = normal(5, 1, 2, T) * level
    Y, dS, dP = run(w, dY)
    ref = oracle_grads(w, dY)
    Y64 = OR.render(w.graph.node_type, w.graph.edges, w.sources, OR.as_params64(w.params)).numpy()
    rP = ref[kind].reshape(dP.shape)
    for c in range(2):
        e = (rel_err(Y[0, c], Y64[0, c]),
             max(rel_err(dS[k, c], ref["S"][k, c]) for k in range(dS.shape[0])),
             grad_err(dP[:, c].reshape(4, -1), rP[:, c].reshape(4, -1)) if left * right > 1e-15 else 0)
        say(f"   channel {c}: Y {e[0]:.2e}, dS {e[1]:.2e}, dP {e[2]:.2e}")
        assert e[0] <= RENDER_TOL and e[1] <= RENDER_TOL and e[2] <= GRAD_TOL, (c, e)


def offsets(w, kind):
    return OP.delay_offsets(w.params[kind][0])  # [2, M]


def reached(mask, offs, sign, half=19):
    """Samples of a channel that a sample set in `mask` [T] enters (sign 1: output of input), within
    `half` taps of each delay."""
    T, out = mask.shape[0], np.zeros(mask.shape[0], bool)
    for d in offs:
        for j in range(-half, half + 1):
            s = sign * (int(d) + j)
            if abs(s) < T:
                out[max(0, s):T + min(0, s)] |= mask[max(0, -s):T - max(0, s)]
    return out


@pytest.mark.parametrize("kind,M", KINDS)
@pytest.mark.parametrize("spans", [([], [(0, 10 ** 9)]), ([(0, 10 ** 9)], []), ([], []),
                                   ([(700, 701)], [(0, 60), (900, 2100)]),
                                   ([(k, k + 1) for k in range(0, 2900, 37)],
                                    [(k, k + 3) for k in range(0, 2900, 41)])])
def test_zeros_stay_exact(kind, M, spans):
    T = 3000 + M * 4410
    say(f"[delay zeros] M={M} spans {spans}")
    w = graph(kind, T, 62, series=False)
    live = np.zeros((2, T), bool)
    for c in range(2):
        for a, b in spans[c]:
            live[c, a:b] = True
    w.sources *= live
    back = live[:, ::-1]
    dY = normal(6, 1, 2, T) * back
    Y, dS, dP = run(w, dY)
    ref = oracle_grads(w, dY)
    Y64 = OR.render(w.graph.node_type, w.graph.edges, w.sources, OR.as_params64(w.params)).numpy()
    offs = offsets(w, kind)
    for c in range(2):
        # the outermost of the 39 taps, j = -19 and 19, are 0
        assert np.all(Y[0, c][~reached(live[c], offs[c], 1, 18)] == 0.0)
        assert np.all(dS[0, c][~reached(back[c], offs[c], -1, 18)] == 0.0)
        assert rel_err(Y[0, c], Y64[0, c]) <= RENDER_TOL
        assert rel_err(dS[0, c], ref["S"][0, c]) <= RENDER_TOL
        if not live[c].any():
            assert np.all(dP[:, c] == 0.0)


@pytest.mark.parametrize("kind,M", KINDS)
@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("channel", [0, 1])
def test_infinities_and_nan_stay_where_they_belong(kind, M, value, channel):
    T = 3000 + M * 4410
    say(f"[delay non-finite] M={M} {value} in channel {channel}")
    w = graph(kind, T, 63, series=False)
    dY = normal(7, 1, 2, T)
    Y0, dS0, dP0 = run(w, dY)
    offs = offsets(w, kind)
    for where in ("input", "adjoint"):
        at = 1234 if where == "input" else T - 1234
        v = graph(kind, T, 63, series=False)
        dV = dY.copy()
        (v.sources if where == "input" else dV)[0, channel, at] = value
        Y, dS, dP = run(v, dV)
        hit = np.zeros(T, bool)
        hit[at] = True
        rows = {"Y": (Y, Y0, 1, where == "input"), "dS": (dS, dS0, -1, where == "adjoint")}
        for name, (got, clean, sign, moved) in rows.items():
            for c in range(2):
                bad = reached(hit, offs[c], sign) & (moved and c == channel)
                assert np.array_equal(~np.isfinite(got[0, c]), bad), (where, name, c)
                assert rel_err(got[0, c][~bad], clean[0, c][~bad]) <= RENDER_TOL, (where, name, c)
        other = 1 - channel
        assert rel_err(dP[0, other], dP0[0, other]) <= RENDER_TOL, where
        # every slot of the channel whose sums hold the value is spoilt
        assert not np.isfinite(dP[0, channel, 0, 2:]).any(), where


@pytest.mark.parametrize("kind,M", KINDS)
def test_values_near_the_largest_float(kind, M):
    """A transform of 512 such values could overflow; their direct sums do not."""
    T = 3000 + M * 4410
    w = graph(kind, T, 64, series=False)
    p = w.params[kind].reshape(-1, 2, M, 22)
    p[..., 2:] = np.minimum(p[..., 2:], -3.0)  # filter gains of 0.05 at most
    w.sources /= np.abs(w.sources).max()
    w.sources[0, 0] *= 3e38
    sched = Schedule(w.graph.node_type, w.graph.edges)
    rb = RenderBuffers(sched, T, with_backward=False)
    rb.forward(torch.as_tensor(w.sources).cuda(),
               {kind: torch.as_tensor(w.params[kind]).cuda()})
    Y = rb.Y.cpu().numpy()
    Y64 = OR.render(w.graph.node_type, w.graph.edges, w.sources, OR.as_params64(w.params)).numpy()
    for c in range(2):
        assert rel_err(Y[0, c], Y64[0, c]) <= RENDER_TOL, c
