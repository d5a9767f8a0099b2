"""Without a native binding that loads (not built, or built for another torch)
the Python functions serve every call through ctypes, as they do what the
binding declines."""

import sys

import numpy as np
import pytest
import torch

from paper_2312_02756_amd import _lib, autograd, glv


@pytest.fixture
def absent(monkeypatch):
    monkeypatch.setattr(_lib, "_native", None)
    monkeypatch.delattr(sys.modules["paper_2312_02756_amd"], "_native", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2312_02756_amd._native", None)  # importing it raises ImportError


def test_it_is_built_here():
    from paper_2312_02756_amd import _native
    assert _lib.native() is _native


def test_calls_reach_the_python_functions(absent):
    c = tuple(torch.ones(4, dtype=torch.float64) for _ in range(4))
    with pytest.warns(RuntimeWarning, match="native binding"):
        with pytest.raises(ValueError, match="GPU tensors"):
            glv.glv_invariant_mass(c, c)
    off = torch.tensor([0, 4])
    for call in (lambda: glv.glv_boost(c, c[:3]), lambda: glv.glv_pair_offsets(off), lambda: glv.glv_event_reduce(c, off),
                 lambda: glv.glv_event_reduce_best_pair(c, off, 91.2), lambda: glv.glv_event_reduce_bwd(c, off),
                 lambda: autograd.invariant_mass(c, c), lambda: autograd.event_reduce(c, off)):
        with pytest.raises(ValueError, match="GPU tensors"):
            call()


@pytest.mark.gpu
def test_results_are_the_same(request):
    import synth
    g = synth.rng(990)
    a, b = (tuple(torch.from_numpy(c).cuda() for c in leg) for leg in synth.pairs_generic(g, 1003))
    off, p = synth.jagged_events(g, 300)
    off, p = torch.from_numpy(off).cuda(), tuple(torch.from_numpy(c).cuda() for c in p)
    leaf = tuple(c.clone().requires_grad_(True) for c in a)

    def calls():
        m = autograd.invariant_mass(leaf, b)
        r = glv.glv_event_reduce(p, off)
        return (m.detach(), *torch.autograd.grad(m, leaf, torch.ones_like(m)), *r[0], *r[1:],
                *glv.glv_event_reduce_bwd(p, off, grad_pair_m=r[2]), *glv.glv_event_reduce_best_pair(p, off, 91.2),
                glv.glv_invariant_mass_histogram(a, b, 0.0, 400.0, 50))

    want = calls()
    request.getfixturevalue("absent")
    with pytest.warns(RuntimeWarning, match="native binding"):
        got = calls()
    for i, (x, y) in enumerate(zip(want, got)):  # NaN: the best mass of an event without pairs
        assert np.array_equal(x.cpu().numpy(), y.cpu().numpy(), equal_nan=True), i


def _forms():
    """Calls that the binding takes, leaves to the Python functions, or that are refused."""
    import synth
    g = synth.rng(991)
    a, b = (tuple(torch.from_numpy(c).cuda() for c in leg) for leg in synth.pairs_generic(g, 300))
    off, p = synth.jagged_events(g, 40)
    off, p = torch.from_numpy(off).cuda(), tuple(torch.from_numpy(c).cuda() for c in p)
    po = glv.glv_pair_offsets(off)
    beta = tuple(0.1 * torch.tanh(c) for c in b[:3])
    one = tuple(c[:1] for c in beta)
    none = tuple(c[:0] for c in a)
    cnt = lambda n, dt=torch.int64: torch.zeros(n, dtype=dt, device="cuda")  # noqa: E731
    mass, hist, red = glv.glv_invariant_mass, glv.glv_invariant_mass_histogram, glv.glv_event_reduce
    best, bwd = glv.glv_event_reduce_best_pair, glv.glv_event_reduce_bwd
    up = torch.ones(int(po[-1]), dtype=torch.float64, device="cuda")
    eye = tuple(torch.full((1,), float(i % 5 == 0), dtype=torch.float64, device="cuda") for i in range(16))
    return [
        lambda: mass(a, b, coords=1), lambda: mass(list(a), torch.stack(b)), lambda: mass(torch.stack(a), b),
        lambda: mass([c.half() for c in a], [c.half() for c in b]), lambda: mass(a[:3], b[:3]),
        lambda: mass(a, [c[:-1] for c in b]), lambda: mass([c[::2] for c in a], [c[::2] for c in b]),
        lambda: mass(a, [c.cpu() for c in b]), lambda: mass(a, b, coords="nowhere"), lambda: mass(none, none),
        lambda: mass(a, b, mode="compensated", fallback_count=cnt(1)), lambda: mass(a, b, fallback_count=cnt(2)),
        lambda: mass(a, b, coords="PxPyPzE", mode="compensated"), lambda: mass([c.requires_grad_(False) for c in a], b),
        lambda: hist(a, b, 0, 400, 50), lambda: hist(a, b, 0.0, 400.0, 0), lambda: hist(a, b, 4.0, 4.0, 10),
        lambda: hist(a, b, 0.0, 400.0, 50, counts=cnt(52)), lambda: hist(a, b, 0.0, 400.0, 50, counts=cnt(50)),
        lambda: hist(a, b, 0.0, 400.0, 50, counts=cnt(52, torch.float64)), lambda: hist(a, b, np.float64(1.0), 400.0, 50),
        lambda: glv.glv_boost(a, beta), lambda: glv.glv_boost(a, one), lambda: glv.glv_boost(a, (*beta[:2], one[0])),
        lambda: glv.glv_boost([c[:1] for c in a], one), lambda: glv.glv_boost(a, beta[:2]),
        lambda: glv.glv_convert(a, 1, 0), lambda: glv.glv_convert(a, "PtEtaPhiM", "PtEtaPhiM"),
        lambda: glv.glv_lorentz_transform(a, eye), lambda: glv.glv_lorentz_transform(a, eye[:15]),
        lambda: glv.glv_rotate_axis_angle(a, eye[:4]), lambda: glv.glv_pair_offsets(off.int()),
        lambda: glv.glv_pair_offsets(off[:1]), lambda: glv.glv_pair_offsets(off[::2]), lambda: red(p, off),
        lambda: red(p, off, po, n_pairs=up.numel()), lambda: red(p, off, want_pair_m=False, want_total=False),
        lambda: red(p, off, mode="compensated", fallback_count=cnt(1)), lambda: red(p, off.int()),
        lambda: red(p, off, po.int()), lambda: red(p, off.cpu()), lambda: red(p, cnt(1)), lambda: red(p, off, n_pairs=-1),
        lambda: red([c.float() for c in p], off, want_total=1), lambda: best(p, off, 91), lambda: best(p, off, "x"),
        lambda: best(p, off, np.float64(91.2), po), lambda: bwd(p, off, grad_pair_m=up), lambda: bwd(p, off, po),
        lambda: bwd(p, off, po, grad_pair_m=up.float()), lambda: bwd(p, off, po, grad_event_m=up[:3]),
        lambda: bwd(p, off, grad_total=[c[:3] for c in p]), lambda: autograd.boost(a, one),
        lambda: autograd.event_reduce(p, off), lambda: autograd.invariant_mass(a, b, mode="other"),
        lambda: autograd.invariant_mass(a, b, coords="PxPyPzE", mode="compensated"),
    ]


def _flat(x):
    return [y for c in x for y in _flat(c)] if isinstance(x, (tuple, list)) else [x]


def _outcome(call):
    try:
        return [t.cpu().numpy() if isinstance(t, torch.Tensor) else t for t in _flat(call())]
    except Exception as e:  # whatever the caller would see
        return type(e)


@pytest.mark.gpu
def test_binding_and_functions_take_and_refuse_the_same(request):
    want = [_outcome(c) for c in _forms()]
    request.getfixturevalue("absent")
    with pytest.warns(RuntimeWarning, match="native binding"):
        got = [_outcome(c) for c in _forms()]
    for i, (x, y) in enumerate(zip(want, got)):
        if isinstance(x, type) or isinstance(y, type):
            assert x is y, (i, x, y)
        else:
            assert len(x) == len(y), i
            for u, v in zip(x, y):
                assert (u is None and v is None) or np.array_equal(u, v, equal_nan=True), i
