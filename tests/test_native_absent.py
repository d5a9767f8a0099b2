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
