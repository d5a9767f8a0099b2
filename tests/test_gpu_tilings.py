"""Which sizes the calls of the Python entry points are launched with."""

import json

import numpy as np
import pytest
import torch

import synth
from gpu_util import gpu
from test_gpu_jagged import _off

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("GLV_AUTOTUNE_CACHE", str(path))
    glv.glv_autotune_forget()
    yield path
    glv.glv_autotune_forget()


def _tune(path, tiling, off, **kw):
    """Makes `tiling` the tuned choice of this process for the events of `off`."""
    key = glv.glv_autotune_key(off, **kw)
    path.write_text(json.dumps({"format": "glv-autotune-1", "entries": [{"key": key, "tiling": list(tiling)}]}))
    assert glv.glv_autotune_lookup(off, **kw) == (tiling, True)


def _events(counts, seed, dtype):
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    g = synth.rng(seed)
    p, _ = synth.pairs_generic(g, int(off[-1]))
    n_pairs = int((counts * (counts - 1) // 2).sum())
    return _off(off), gpu(p, dtype), gpu([g.standard_normal(n_pairs)], dtype)[0]


def test_tuned_reverse_mode_is_taken_also_where_it_equals_the_default(cache):
    """Events of 40 particles: 780 pairs, more than the default stages, so
    that the launch they are done in, and the order of their sums, tells the
    sizes apart."""
    off, p, up = _events(np.full(400, 40), 980, torch.float32)
    po = glv.glv_pair_offsets(off)
    run = lambda t: glv.glv_event_reduce_bwd(p, off, po, grad_pair_m=up, tiling=t)  # noqa: E731
    default = (128, 64, 128, 512)
    want, untuned = run(default), run(None)
    assert not all(torch.equal(a, b) for a, b in zip(untuned, want))
    _tune(cache, default, off, dtype=torch.float32, backward=True)
    assert all(torch.equal(a, b) for a, b in zip(run(None), want))
    leaves = tuple(c.clone().requires_grad_(True) for c in p)
    from paper_2312_02756_amd import autograd as ag
    pm = ag.event_reduce(leaves, off, po)[2]
    assert all(torch.equal(a, b) for a, b in zip(torch.autograd.grad(pm, leaves, up), want))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_every_route_takes_the_same_sizes(dtype):
    """The native binding, the Python functions behind it and a C call given
    glv_call_tiling's sizes: the same gradients, bit for bit."""
    glv.glv_autotune_forget()
    for mean in (5, 12, 20, 40, 60):
        counts = synth.rng(981 + mean).poisson(mean, 3000)
        off, p, up = _events(counts, 982 + mean, dtype)
        po = glv.glv_pair_offsets(off)
        t = glv.glv_call_tiling(3000, up.numel(), dtype, backward=True)
        want = glv.glv_event_reduce_bwd(p, off, po, grad_pair_m=up, tiling=t)
        native = glv.glv_event_reduce_bwd(p, off, po, grad_pair_m=up)
        python = glv.glv_event_reduce_bwd(p, off, po, grad_pair_m=up, coords=1)  # declined by the binding
        assert all(torch.equal(a, b) and torch.equal(a, c) for a, b, c in zip(want, native, python))


@pytest.mark.parametrize("backward", [False, True])
def test_a_miss_drops_the_choice_made_for_other_events(cache, backward):
    off, _, _ = _events(np.full(400, 40), 983, torch.float64)
    other, _, _ = _events(np.full(400, 5), 984, torch.float64)
    untuned = glv.glv_call_tiling(400, 400 * 10, backward=backward)
    _tune(cache, (64, 16, 64, 256), off, backward=backward)
    assert glv.glv_call_tiling(400, 400 * 10, backward=backward) == (64, 16, 64, 256)
    assert glv.glv_autotune_lookup(other, backward=backward)[1] is False
    assert glv.glv_call_tiling(400, 400 * 10, backward=backward) == untuned
    assert glv.glv_autotune_lookup(off, backward=backward) == ((64, 16, 64, 256), True)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_autotuning_tries_what_an_untuned_call_takes(cache, dtype):
    """1,000 events of 22 particles: tiles of four events, which only the
    untuned choice has, spread them over several times as much of the GPU as
    the smallest of the other candidates (16)."""
    cache.unlink(missing_ok=True)
    off, p, up = _events(np.full(1000, 22), 985, dtype)
    assert glv.glv_autotune_event_reduce(p, off) == glv.glv_current_tiling(dtype)
    assert glv.glv_current_tiling(dtype)[1] == 4
    best = glv.glv_autotune_event_reduce_bwd(p, off, grad_pair_m=up)
    assert best == glv.glv_current_tiling_bwd(dtype) and best[1] == 4


@pytest.mark.parametrize("mode", ["plain", "compensated"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_untuned_best_pair_is_no_slower_than_given_sizes(mode, dtype):
    """2^18 events of 8 particles: the sizes of an untuned call against those
    calls took before they followed type and mode (a third more time in the
    FP32 compensated mode at the plain one's sizes), with room for noise."""
    glv.glv_autotune_forget()
    off, p, _ = _events(synth.rng(986).poisson(8.0, 1 << 18), 987, dtype)
    po = glv.glv_pair_offsets(off)

    def us(tiling):
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        ev[0].record()
        for _ in range(5):
            glv.glv_event_reduce_best_pair(p, off, 91.2, po, mode=mode, tiling=tiling)
        ev[1].record()
        ev[1].synchronize()
        return ev[0].elapsed_time(ev[1]) * 200.0

    us((0, 0, 0, 0)), us((64, 64, 128, 1024))
    turns = [(us((0, 0, 0, 0)), us((64, 64, 128, 1024))) for _ in range(9)]
    untuned, given = (sorted(t[k] for t in turns)[4] for k in (0, 1))
    assert untuned < 1.1 * given, (untuned, given)
