"""GPU parity of the batched render and its adjoint against the FP64 oracle (paper Algorithm 1;
processors of Sec. 3). Sizes span several tiles with ragged tails (T % 2048 != 0, both T % 4 == 0
and T % 4 != 0) so every kernel's edge handling runs."""
import numpy as np
import pytest
import torch

import synth
from gpu_common import (GRAD_TOL, check_render, device_inputs, grad_err, oracle_grads,
                        rel_err, say)
from paper_2408_03204_amd import RenderBuffers, Schedule, merge_graphs, render

pytestmark = pytest.mark.gpu

T_RAGGED = [3 * 2048 + 555, 4 * 2048 + 1024 + 4]
SINGLE_TYPES = [synth.MIX, synth.GAIN_PAN, synth.IMAGER, synth.TANH, synth.EQ, synth.COMP,
                synth.DELAY]


def single_node_workload(t, T, seed):
    b = synth.GraphBuilder()
    i0, i1 = b.add(synth.IN), b.add(synth.IN)
    n = b.add(t)
    o = b.add(synth.OUT)
    b.connect(i0, n)
    b.connect(i1, n)
    b.connect(i0, n)  # parallel edge: counted twice
    b.connect(n, o)
    g = b.build()
    return synth.Workload(f"single_{t}", g, synth.make_sources(synth.rng_for(seed, 1), 2, T),
                          synth.draw_params(synth.rng_for(seed, 2), g), None, T, seed)


@pytest.mark.parametrize("T", T_RAGGED)
@pytest.mark.parametrize("t", SINGLE_TYPES)
def test_single_processor_forward(t, T):
    say(f"[single fwd] type={t} T={T}")
    w = single_node_workload(t, T, 10 + t)
    sched = Schedule(w.graph.node_type, w.graph.edges)
    S, P = device_inputs(w)
    Y, U = render(sched, S, P, return_U=True)
    torch.cuda.synchronize()
    check_render(w, sched, Y, U)


@pytest.mark.parametrize("seed", range(4))
def test_random_dag_forward(seed):
    T = T_RAGGED[seed % 2]
    say(f"[random fwd] seed={seed} T={T}")
    w = synth.random_workload(500 + seed, 14, T, edge_p=0.3, n_out=1 + seed % 2)
    sched = Schedule(w.graph.node_type, w.graph.edges)
    S, P = device_inputs(w)
    Y, U = render(sched, S, P, return_U=True)
    torch.cuda.synchronize()
    check_render(w, sched, Y, U)


def test_tiny_console_forward():
    say("[tiny console fwd] T=2^15")
    w = synth.tiny_console(T=2 ** 15)
    sched = Schedule(w.graph.node_type, w.graph.edges)
    S, P = device_inputs(w)
    Y, U = render(sched, S, P, return_U=True)
    torch.cuda.synchronize()
    check_render(w, sched, Y, U)


def test_schedule_invariance_and_determinism():
    """All four schedules give bit-identical renders (each node's arithmetic is fixed), and two
    runs give identical bits."""
    say("[invariance] random dag, 4 methods")
    w = synth.random_workload(77, 12, 5 * 2048 + 77, edge_p=0.35)
    S, P = device_inputs(w)
    ref = None
    for m in ("one_by_one", "greedy", "beam", "optimal"):
        sched = Schedule(w.graph.node_type, w.graph.edges, m)
        Y = render(sched, S, P)
        torch.cuda.synchronize()
        if ref is None:
            ref = Y.clone()
            Y2 = render(sched, S, P)
            assert torch.equal(Y2, ref)
        else:
            assert torch.equal(Y, ref), m


def test_empty_and_trivial_graphs():
    say("[trivial] in->out, orphan processor, T=1 and T=5")
    for T in (1, 5, 2048):
        g = synth.Graph(np.array([0, 3, 1, 1, 0], dtype=np.int32),
                        np.array([[0, 0, 1], [2, 1, 3]], dtype=np.int32))
        w = synth.Workload("trivial", g, synth.make_sources(synth.rng_for(1, 1), 2, T),
                           synth.draw_params(synth.rng_for(1, 2), g), None, T, 1)
        sched = Schedule(g.node_type, g.edges)
        S, P = device_inputs(w)
        Y, U = render(sched, S, P, return_U=True)
        torch.cuda.synchronize()
        check_render(w, sched, Y, U)


@pytest.mark.parametrize("T", [3, 1023, 1025, 4096 + 1022])
def test_pointwise_odd_lengths(T):
    """Rows that do not start on 16-byte boundaries, with one, two and three samples past the last
    whole group and a last tile of one sample: forward and adjoint of a gain, imager and tanh
    chain against the oracle (the usual tolerances)."""
    say(f"[pointwise odd] T={T}")
    b = synth.GraphBuilder()
    i0, i1 = b.add(synth.IN), b.add(synth.IN)
    a, z = b.chain([synth.GAIN_PAN, synth.IMAGER, synth.TANH, synth.MIX, synth.OUT])
    b.connect(i0, a)
    b.connect(i1, a)
    g = b.build()
    w = synth.Workload("odd", g, synth.make_sources(synth.rng_for(7, 1), 2, T),
                       synth.draw_params(synth.rng_for(7, 2), g), None, T, 7)
    sched = Schedule(g.node_type, g.edges)
    S, P = device_inputs(w)
    Y, U = render(sched, S, P, return_U=True)
    torch.cuda.synchronize()
    check_render(w, sched, Y, U)
    for k, e in run_backward(w, 8).items():
        assert e <= GRAD_TOL, (k, e)


@pytest.mark.parametrize("n", [1, 16, 17, 33])
def test_eq_node_counts(n):
    """EQ designs and parameter gradients around the 16 nodes that one block of the design products
    takes, forward and adjoint against the oracle (the usual tolerances), and to the bit against
    each node rendered alone."""
    T = 2048 + 77
    say(f"[eq nodes] n={n}")
    b = synth.GraphBuilder()
    for _ in range(n):
        i, e, o = b.add(synth.IN), b.add(synth.EQ), b.add(synth.OUT)
        b.connect(i, e)
        b.connect(e, o)
    g = b.build()
    w = synth.Workload("eqs", g, synth.make_sources(synth.rng_for(n, 1), n, T),
                       synth.draw_params(synth.rng_for(n, 2), g), None, T, n)
    sched = Schedule(g.node_type, g.edges)
    S, P = device_inputs(w)
    Y, U = render(sched, S, P, return_U=True)
    torch.cuda.synchronize()
    check_render(w, sched, Y, U)
    for k, e in run_backward(w, n).items():
        assert e <= GRAD_TOL, (k, e)
    one = synth.GraphBuilder()
    one.chain([synth.IN, synth.EQ, synth.OUT])
    g1 = one.build()
    s1 = Schedule(g1.node_type, g1.edges)
    for k in {0, n // 2, n - 1}:
        y = render(s1, S[k:k + 1].clone(), {synth.EQ: P[synth.EQ][k:k + 1].clone()})
        assert torch.equal(y[0], Y[k]), k


# ---- adjoint -------------------------------------------------------------------------------


def run_backward(w, seed):
    sched = Schedule(w.graph.node_type, w.graph.edges)
    S, P = device_inputs(w)
    S.requires_grad_(True)
    for p in P.values():
        p.requires_grad_(True)
    Y = render(sched, S, P)
    dY = np.random.default_rng(seed).normal(size=tuple(Y.shape)).astype(np.float32)
    Y.backward(torch.as_tensor(dY).cuda())
    torch.cuda.synchronize()
    ref = oracle_grads(w, dY)
    errs = {"S": grad_err(S.grad.cpu().numpy(), ref["S"])}
    for t, p in P.items():
        errs[t] = grad_err(p.grad.cpu().numpy(), ref[t])
    return errs


@pytest.mark.parametrize("T", T_RAGGED)
@pytest.mark.parametrize("t", SINGLE_TYPES)
def test_single_processor_backward(t, T):
    say(f"[single bwd] type={t} T={T}")
    w = single_node_workload(t, T, 30 + t)
    errs = run_backward(w, t)
    say("   grad errs", errs)
    for k, e in errs.items():
        assert e <= GRAD_TOL, (k, e)


@pytest.mark.parametrize("seed", range(4))
def test_random_dag_backward(seed):
    T = T_RAGGED[seed % 2]
    say(f"[random bwd] seed={seed} T={T}")
    w = synth.random_workload(600 + seed, 14, T, edge_p=0.3, n_out=1 + seed % 2)
    errs = run_backward(w, seed)
    say("   grad errs", errs)
    for k, e in errs.items():
        assert e <= GRAD_TOL, (k, e)


def test_tiny_console_backward():
    say("[tiny console bwd]")
    errs = run_backward(synth.tiny_console(T=2 ** 15), 3)
    say("   grad errs", errs)
    for k, e in errs.items():
        assert e <= GRAD_TOL, (k, e)


@pytest.mark.parametrize("a", [0.0, 0.999999])
def test_compressor_alpha_edge_values(a):
    """alpha at the ends of its domain [0, 1): 0 (no smoothing, g = x) and a time constant of
    about 23 s, across several 3072-sample chunks, forward and adjoint against the oracle. With
    a = 0 the chunk carry weights A^d (A = a^3072) must be 1 for the adjacent chunk and 0 beyond;
    near 1 every earlier chunk's total reaches the carry."""
    T = 5 * 3072 + 77
    say(f"[compressor alpha={a}] T={T}")
    w = single_node_workload(synth.COMP, T, 41)
    w.params[synth.COMP][:, 0] = a
    sched = Schedule(w.graph.node_type, w.graph.edges)
    S, P = device_inputs(w)
    Y, U = render(sched, S, P, return_U=True)
    torch.cuda.synchronize()
    check_render(w, sched, Y, U)
    errs = run_backward(w, 5)
    say("   grad errs", errs)
    for k, e in errs.items():
        assert e <= GRAD_TOL, (k, e)


@pytest.mark.parametrize("unroll", [1, 2, 4])
@pytest.mark.parametrize("T", [3, 1025, 2 * 4096 + 4])
def test_pointwise_chains(T, unroll):
    """Runs of pointwise steps whose nodes form paths are one launch, up to four steps at a time:
    paths of five nodes (a tanh first, so the adjoint needs the sources; another inside), then a
    mix -> gain -> out path. Output rows and input adjoints equal the single steps' to the bit;
    everything equals the oracle to the usual tolerances."""
    say(f"[pointwise chains] T={T} unroll={unroll}")
    b = synth.GraphBuilder()
    ends = []
    for _ in range(3):
        ends.append(b.chain([synth.IN, synth.TANH, synth.GAIN_PAN, synth.IMAGER, synth.TANH,
                             synth.GAIN_PAN])[1])
    a, _ = b.chain([synth.MIX, synth.GAIN_PAN, synth.OUT])
    for v in ends:
        b.connect(v, a)
    g = b.build()
    S = synth.make_sources(synth.rng_for(3, 1), 3, T)
    S[0, :, ::3] = -0.0
    w = synth.Workload("chains", g, S, synth.draw_params(synth.rng_for(3, 2), g), None, T, 3)
    sched = Schedule(g.node_type, g.edges)
    sched.set_tuning(Schedule.TUNE_POINTWISE_UNROLL, unroll)
    Sd, P = device_inputs(w)
    buf = RenderBuffers(sched, T, "cuda")
    dY = torch.as_tensor(np.random.default_rng(4).normal(size=tuple(buf.Y.shape))
                         .astype(np.float32)).cuda()
    dS, dP = torch.empty_like(Sd), {t: torch.empty_like(p) for t, p in P.items()}
    buf.U.fill_(7.0)
    buf.dU.fill_(7.0)
    buf.forward(Sd, P)
    buf.backward(Sd, P, dY, dP, dS)
    U, dU = buf.U.clone(), buf.dU.clone()
    buf.U.fill_(7.0)
    buf.dU.fill_(7.0)
    for n in range(1, sched.num_steps + 1):
        buf.step(Sd, P, n)
    for n in range(sched.num_steps - 1, 0, -1):
        buf.backward_step(Sd, P, dY, n)
    torch.cuda.synchronize()
    assert torch.equal(U.view(torch.int32), buf.U.view(torch.int32))
    assert torch.equal(dU.view(torch.int32), buf.dU.view(torch.int32))
    check_render(w, sched, U[sched.out_begin:], U)
    ref = oracle_grads(w, dY.cpu().numpy())
    assert grad_err(dS.cpu().numpy(), ref["S"]) <= GRAD_TOL
    for t, p in dP.items():
        assert grad_err(p.cpu().numpy(), ref[t]) <= GRAD_TOL, t


@pytest.mark.parametrize("L", [5, 2048 * 3 + 1, 2048 * 32, 2048 * 32 + 1])
def test_eq_gradients_alone_and_merged(L):
    """An EQ's parameter gradient is the same bits whether its cross-spectra are summed by the
    transform's launch (rows of up to 32 tiles) or by a launch of their own, as in a graph merged
    with a longer one; a gain's reduction rides along in either."""
    say(f"[eq gradients] L={L}")

    def graph():
        b = synth.GraphBuilder()
        b.chain([synth.IN, synth.EQ, synth.GAIN_PAN, synth.OUT])
        return b.build()

    g, lens = graph(), [L, 2048 * 33 + 7]
    m = merge_graphs([(g.node_type, g.edges, n) for n in lens])
    rng = np.random.default_rng(L)
    P = {synth.EQ: torch.as_tensor(rng.normal(0, 0.5, (2, 1024)).astype(np.float32)).cuda(),
         synth.GAIN_PAN: torch.as_tensor(rng.normal(0, 0.5, (2, 2)).astype(np.float32)).cuda()}
    S = torch.zeros((2, 2, m["T"]), device="cuda")
    dY = torch.zeros_like(S)
    for i, n in enumerate(lens):
        S[i, :, :n] = torch.as_tensor(rng.normal(size=(2, n)).astype(np.float32))
        dY[i, :, :n] = torch.as_tensor(rng.normal(size=(2, n)).astype(np.float32))
    grads = []
    for nodes, edges, lengths, T, rows in ((m["node_type"], m["edges"], m["lengths"], m["T"], 2),
                                           (g.node_type, g.edges, None, L, 1)):
        sched = Schedule(nodes, edges, lengths=lengths)
        buf = RenderBuffers(sched, T, "cuda")
        Pr = {t: p[:rows].clone() for t, p in P.items()}
        dP = {t: torch.empty_like(p) for t, p in Pr.items()}
        s = S[:rows, :, :T].clone(memory_format=torch.contiguous_format)
        d = dY[:rows, :, :T].clone(memory_format=torch.contiguous_format)
        buf.forward(s, Pr)
        buf.backward(s, Pr, d, dP)
        torch.cuda.synchronize()
        grads.append({t: p[0] for t, p in dP.items()})
    for t in P:
        assert torch.equal(grads[0][t], grads[1][t]), t


@pytest.mark.parametrize("lone", [True, False])
@pytest.mark.parametrize("T", [777, 4096 + 1030])
@pytest.mark.parametrize("t", sorted(set(range(2, 13))))
def test_source_adjoints(t, T, lone):
    """Where every source is one processor's only input, the processors' kernels store the source
    adjoints, otherwise (several consumers, parallel edges, straight to an output, a consumer with
    two inputs) the input step does: every row is the sum of its consumers' adjoint rows in edge
    order, to the bit, for every node type."""
    say(f"[source adjoints] type={t} T={T} lone={lone}")
    b = synth.GraphBuilder()
    ins = [b.add(synth.IN) for _ in range(3 if lone else 6)]
    nodes = [b.add(t) for _ in range(3 if lone else 4)]
    o = b.add(synth.OUT)
    edges = [(0, 1), (1, 0), (2, 2)]
    if not lone:
        edges += [(2, 2), (3, 1), (4, None), (4, 0), (5, 3)]
    for x, y in edges:
        b.connect(ins[x], o if y is None else nodes[y])
    for v in nodes:
        b.connect(v, o)
    g = b.build()
    K = len(ins)
    w = synth.Workload("sources", g, synth.make_sources(synth.rng_for(t, 1), K, T),
                       synth.draw_params(synth.rng_for(t, 2), g), None, T, t)
    sched = Schedule(g.node_type, g.edges)
    S, P = device_inputs(w)
    if t == synth.REVERB:
        sched.set_reverb_noise(torch.rand((2, 3000), device="cuda") - 0.5)
    buf = RenderBuffers(sched, T, "cuda")
    dY = torch.as_tensor(np.random.default_rng(t).normal(size=tuple(buf.Y.shape))
                         .astype(np.float32)).cuda()
    dS = torch.full_like(S, 7.0)
    buf.forward(S, P)
    buf.backward(S, P, dY, {k: torch.empty_like(p) for k, p in P.items()}, dS)
    torch.cuda.synchronize()
    for k in range(K):
        ref = torch.zeros_like(dS[k])
        for v in sched.out_dst[sched.out_ptr[k]:sched.out_ptr[k + 1]]:
            ref = ref + (dY[v - sched.out_begin] if v >= sched.out_begin else buf.dU[int(v)])
        assert torch.equal(dS[k].view(torch.int32), ref.view(torch.int32)), k


@pytest.mark.parametrize("L", [2048 * 16, 2048 * 16 + 1])
def test_eq_gradients_on_either_side_of_the_fold(L):
    """The longest rows whose cross-spectra the transform's launch sums (16 tiles) and the shortest that
    have a launch of their own (17): the same bits as in a graph merged with a longer one."""
    test_eq_gradients_alone_and_merged(L)
