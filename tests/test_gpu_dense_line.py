"""Events of the mean sizes around which the jagged reduction's second launch
takes all but the smallest, on either side of the numbers of events where that
line changes."""

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import gpu
from test_gpu_jagged import _check_forward, _off

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")


def _events(ne, mean, seed):
    g = synth.rng(seed)
    counts = g.poisson(mean, ne)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    p, _ = synth.pairs_generic(g, int(off[-1]))
    return off, p


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("mode,means", [("plain", (24, 27)), ("compensated", (17, 19, 23))])
@pytest.mark.parametrize("ne", [4096, 4097])
def test_masses_around_the_lines(ne, mode, means, dtype):
    for mean in means:
        off, p = _events(ne, mean, 840 + mean)
        pg, og = gpu(p, dtype), _off(off)
        total, em, pm = glv.glv_event_reduce(pg, og, mode=mode)
        _check_forward(off, p, dtype, "PtEtaPhiM", mode, total, em, pm, f"{ne} {mean} {mode} {dtype}")


@pytest.mark.parametrize("ne", [49152, 49153, (1 << 18) - 1, 1 << 18])
def test_best_pair_around_the_lines(ne):
    """Events of 31 to 33 particles, 496 pairs on average: in the second launch
    up to 49,152 events, in the first beyond; the pair selected from stored masses."""
    off = np.concatenate([[0], np.cumsum(31 + np.arange(ne) % 3)]).astype(np.int64)
    n, n_pairs = int(off[-1]), int(oracle.pair_offsets(off)[-1])
    gen = torch.Generator(device="cuda")
    gen.manual_seed(850)
    p = [torch.rand(n, device="cuda", generator=gen) for _ in range(4)]
    p = (p[0] * 95 + 5, p[1] * 5 - 2.5, p[2] * 6.2 - 3.1, p[3] * 0.2)
    og = _off(off)
    po = glv.glv_pair_offsets(og)
    rank, bm = glv.glv_event_reduce_best_pair(p, og, 91.2, po)
    pm = glv.glv_event_reduce(p, og, po, n_pairs=n_pairs)[2]
    want_r, want_m = glv.glv_event_best_pair(po, pm, 91.2)
    assert torch.equal(rank, want_r) and torch.equal(bm, want_m)
