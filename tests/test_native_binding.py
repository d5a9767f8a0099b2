"""The native part of the binding: it declines (returns None for) whatever is
not a plain call, so that the Python path decides, and its autograd nodes do
what the Python classes do."""

import threading

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2312_02756_amd import _lib

gpu_test = pytest.mark.gpu


def _cpu_calls():
    c = tuple(torch.ones(4, dtype=torch.float64) for _ in range(4))
    off = torch.tensor([0, 4])
    return [("mass", (c, c, "PtEtaPhiM", "plain", None)), ("mass", (c[:3], c, "PtEtaPhiM", "plain", None)),
            ("mass", (None, c, "PtEtaPhiM", "plain", None)), ("mass", (iter(c), c, "PtEtaPhiM", "plain", None)),
            ("mass", ()), ("mass_histogram", (c, c, 0.0, 1.0, 10, "PtEtaPhiM", "plain", None, None)),
            ("boost", (c, c[:3])), ("convert", (c, "PtEtaPhiM", "PxPyPzE")), ("convert", (c, 1, 0)),
            ("transform", (c, c)), ("transform", (c, ())), ("pair_offsets", (off,)), ("pair_offsets", ([0, 4],)),
            ("event_reduce", (c, off, None, "PtEtaPhiM", "plain", True, True, True, None, None)),
            ("event_reduce_best_pair", (c, off, 91.2, None, "PtEtaPhiM", "plain", None)),
            ("autograd_mass", (c, c, "PtEtaPhiM", "plain")), ("autograd_boost", (c, c[:3])),
            ("autograd_event_reduce", (c, off, None, "PtEtaPhiM"))]


@pytest.mark.parametrize("i", range(len(_cpu_calls())))
def test_declines_what_is_no_plain_gpu_call(i):
    fn, args = _cpu_calls()[i]
    assert getattr(_lib.native(), fn)(*args) is None


def _legs(n, seed, dtype=torch.float64):
    g = synth.rng(seed)
    a, b = synth.pairs_generic(g, n)
    up = torch.from_numpy(g.standard_normal(n))
    return [tuple(torch.from_numpy(c).cuda().to(dtype) for c in leg) for leg in (a, b)] + [up.cuda().to(dtype)]


def _events(ne, seed):
    off, p = synth.jagged_events(synth.rng(seed), ne)
    return torch.from_numpy(off).cuda(), tuple(torch.from_numpy(c).cuda() for c in p)


def _leaves(cols):
    return tuple(c.detach().clone().requires_grad_(True) for c in cols)


@gpu_test
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("mode", ["plain", "compensated"])
def test_nodes_match_the_python_classes(mode, dtype):
    """Outputs and gradients bitwise those of the Python classes; unused outputs give zeros."""
    from paper_2312_02756_amd import autograd as ag, glv
    a, b, up = _legs(1003, 950, dtype)
    for apply in (lambda x, y: ag.invariant_mass(list(x), y, mode=mode),
                  lambda x, y: ag.InvariantMass.apply("PtEtaPhiM", mode, *x, *y)):
        la, lb = _leaves(a), _leaves(b)
        m = apply(la, lb)
        g = torch.autograd.grad(m, (*la, *lb), up)
        if "first" not in locals():
            first = (m.detach(), *g)
    assert all(torch.equal(x, y) for x, y in zip(first, (m, *g)))
    beta = tuple(0.3 * torch.tanh(c) for c in b[:3])
    got = []
    for apply in (ag.boost, lambda x, y: ag.Boost.apply(*x, *y)):
        lx, lb = _leaves(a), _leaves(beta)
        y = apply(lx, lb)
        got.append((*(c.detach() for c in y), *torch.autograd.grad(y[1:3], (*lx, *lb), (up, 2 * up))))
    assert all(torch.equal(x, y) for x, y in zip(*got))
    off, p = _events(300, 951)
    p = tuple(c.to(dtype) for c in p)
    got = []
    for po in (None, glv.glv_pair_offsets(off)):
        for apply in (lambda q: ag.event_reduce(q, off, po),
                      lambda q: (lambda o: (o[:4], o[4], o[5]))(
                          ag.EventReduce.apply(off, glv.glv_pair_offsets(off), "PtEtaPhiM", *q))):
            q = _leaves(p)
            total, em, pm = apply(q)
            got.append((em.detach(), *torch.autograd.grad((total[3], pm), q, (torch.ones_like(em), pm.detach()))))
    assert all(torch.equal(x, y) for o in got[1:] for x, y in zip(got[0], o))


@gpu_test
def test_hooks_versions_and_transforms():
    """Saved-tensor hooks see every saved column, changed saved columns are
    refused, and forward mode and functorch are refused as by the classes."""
    from paper_2312_02756_amd import autograd as ag
    a, b, up = _legs(64, 952)
    la, lb = _leaves(a), _leaves(b)
    seen = []
    with torch.autograd.graph.saved_tensors_hooks(lambda t: seen.append(1) or t.cpu(), lambda t: t.cuda()):
        m = ag.invariant_mass(la, lb)
    assert len(seen) == 8
    want = torch.autograd.grad(ag.invariant_mass(la, lb), la, up)
    assert all(torch.equal(x, y) for x, y in zip(torch.autograd.grad(m, la, up), want))
    m = ag.invariant_mass(la, lb)
    with torch.no_grad():
        la[0].add_(1.0)
    with pytest.raises(RuntimeError, match="modified by an inplace operation"):
        m.backward(up)
    with torch.autograd.forward_ad.dual_level():
        d = (torch.autograd.forward_ad.make_dual(a[0], up), *a[1:])
        with pytest.raises(RuntimeError):
            ag.invariant_mass(d, b)
    with pytest.raises(RuntimeError):
        torch.func.vmap(lambda x: ag.invariant_mass((x, *a[1:]), b))(torch.stack([a[0], a[0]]))


@gpu_test
def test_errors_are_those_of_the_python_path():
    from paper_2312_02756_amd import glv
    a, b, _ = _legs(64, 953)
    with pytest.raises(ValueError):
        glv.glv_invariant_mass(a, tuple(c.float() for c in b))
    with pytest.raises(ValueError):
        glv.glv_invariant_mass(a, tuple(c[:-1] for c in b))
    with pytest.raises(_lib.GlvError):
        glv.glv_invariant_mass(a, b, coords="PxPyPzE", mode="compensated")
    with pytest.raises(_lib.GlvError):
        glv.glv_invariant_mass_histogram(a, b, 1.0, 1.0, 10)
    with pytest.raises(KeyError):
        glv.glv_convert(a, "PtEtaPhiM", "nowhere")


@gpu_test
def test_threads_and_streams():
    """Calls from several threads, each on a stream of its own."""
    from paper_2312_02756_amd import autograd as ag, glv
    off, p = _events(2000, 954)
    a, b, up = _legs(20000, 955)
    want = (glv.glv_event_reduce(p, off)[2], glv.glv_invariant_mass(a, b))
    torch.cuda.synchronize()
    bad = []

    def work():
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                la = _leaves(a)
                m = ag.invariant_mass(la, b)
                g = torch.autograd.grad(m, la, up)
                pm = glv.glv_event_reduce(p, off)[2]
                if not (torch.equal(pm, want[0]) and torch.equal(m, want[1]) and all(torch.isfinite(c).all() for c in g)):
                    bad.append(1)

    ts = [threading.Thread(target=work) for _ in range(4)]
    [t.start() for t in ts]
    [t.join() for t in ts]
    assert not bad


@gpu_test
def test_capture():
    """The calls in a captured graph, replayed after new inputs."""
    from paper_2312_02756_amd import glv
    off, p = _events(5000, 956)
    a, b, _ = _legs(5000, 957)
    n_pairs = int(oracle.pair_offsets(off.cpu().numpy())[-1])

    def calls():
        return (glv.glv_invariant_mass(a, b), glv.glv_event_reduce(p, off, n_pairs=n_pairs)[2],
                *glv.glv_event_reduce_best_pair(p, off, 91.2),
                glv.glv_invariant_mass_histogram(a, b, 0.0, 400.0, 100))

    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        calls()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        out = calls()
    for k in range(3):
        for c in (a[0], p[0]):
            c.mul_(1.0 + 0.1 * k)
        g.replay()
        torch.cuda.synchronize()
        for x, y in zip(out, calls()):
            np.testing.assert_array_equal(x.cpu().numpy(), y.cpu().numpy())
