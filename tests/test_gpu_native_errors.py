"""A library call that reports an error of the HIP runtime raises once and is
not made again: what it added to the caller's counters stays added once.  The
error is a pending one, left by a refused hipSetDevice, which the next launch's
check reports although the kernel itself runs."""

import ctypes

import pytest
import torch

import synth
from paper_2312_02756_amd import _lib

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")


def _pending_error():
    hip = ctypes.CDLL("libamdhip64.so.7")  # the runtime this process has loaded
    assert hip.hipSetDevice(1 << 20) != 0


def _legs(n, seed, dtype):
    a, b = synth.pairs_generic(synth.rng(seed), n)
    return [tuple(torch.from_numpy(c).cuda().to(dtype) for c in leg) for leg in (a, b)]


def test_given_counts_are_added_once():
    a, b = _legs(5000, 970, torch.float64)
    want = glv.glv_invariant_mass_histogram(a, b, 0.0, 400.0, 50)
    counts = torch.zeros_like(want)
    torch.cuda.synchronize()
    _pending_error()
    with pytest.raises(_lib.GlvError) as e:
        glv.glv_invariant_mass_histogram(a, b, 0.0, 400.0, 50, counts=counts)
    assert e.value.code == 10
    torch.cuda.synchronize()
    assert torch.equal(counts, want)
    # the next call is a new one
    assert torch.equal(glv.glv_invariant_mass_histogram(a, b, 0.0, 400.0, 50), want)


def test_errors_of_allocation_and_filling_raise():
    a, b = _legs(300, 973, torch.float64)
    glv.glv_invariant_mass_histogram(a, b, 0.0, 400.0, 50)
    torch.cuda.synchronize()
    _pending_error()
    with pytest.raises(RuntimeError):  # torch's own, from the counters' zeroing
        glv.glv_invariant_mass_histogram(a, b, 0.0, 400.0, 50)


def test_calls_and_nodes_raise():
    from paper_2312_02756_amd import autograd as ag
    a, b = _legs(300, 971, torch.float64)
    off, p = synth.jagged_events(synth.rng(972), 200)
    off, p = torch.from_numpy(off).cuda(), tuple(torch.from_numpy(c).cuda() for c in p)
    beta = tuple(0.1 * torch.tanh(c) for c in b[:3])
    po = glv.glv_pair_offsets(off)
    leaf = tuple(c.clone().requires_grad_(True) for c in a)
    n_pairs = int(po[-1])
    up = torch.ones_like(a[0])
    calls = [lambda: glv.glv_invariant_mass(a, b), lambda: glv.glv_boost(a, beta), lambda: glv.glv_pair_offsets(off),
             lambda: glv.glv_convert(a, "PtEtaPhiM", "PxPyPzE"),
             lambda: glv.glv_event_reduce(p, off, po, n_pairs=n_pairs),
             lambda: glv.glv_event_reduce_best_pair(p, off, 91.2, po),
             lambda: ag.invariant_mass(leaf, b), lambda: ag.boost(leaf, beta)]
    for k, call in enumerate(calls):
        call()  # its memory is at hand from here on
        torch.cuda.synchronize()
        _pending_error()
        with pytest.raises(_lib.GlvError):
            call()
            pytest.fail(f"call {k}")
        call()
    # no gradient node is left half done
    assert all(torch.isfinite(g).all() for g in torch.autograd.grad(ag.invariant_mass(leaf, b), leaf, up))
