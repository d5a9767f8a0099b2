"""Large events far from where equal events would put a workgroup's share of the
pairs, at the numbers of events where the windows of the large-event launches
change: all of them in one window or not, one slice or several, few pairs or
many."""

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import gpu
from test_gpu_jagged import _off

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")

LARGE = np.array([60, 300, 49, 97, 1000, 64, 130, 200], dtype=np.int64)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("where", ["first", "middle", "last", "alone"])
@pytest.mark.parametrize("ne", [2048, 2049, 3072, 3073, 4096, 4097, 5000, 20000, 200000])
def test_large_events_away_from_their_place(ne, where, dtype):
    """Bitwise the results of the large events in a call of their own, in which
    the workgroups' shares of the reverse mode differ; "alone" has no pairs
    elsewhere, so that the shares are as small as they get."""
    g = synth.rng(860)
    counts = g.integers(0, 2, ne) if where == "alone" else g.poisson(8, ne)
    at = {"first": 3, "middle": ne // 3, "last": ne - len(LARGE), "alone": ne - 700}[where] + np.arange(len(LARGE))
    counts[at] = LARGE
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    own = np.concatenate([[0], np.cumsum(LARGE)]).astype(np.int64)
    po = oracle.pair_offsets(off)
    p, _ = synth.pairs_generic(g, int(off[-1]))
    rows = slice(int(off[at[0]]), int(off[at[-1] + 1]))
    pairs = slice(int(po[at[0]]), int(po[at[-1] + 1]))
    ev = slice(int(at[0]), int(at[-1] + 1))
    pg, og = gpu(p, dtype), _off(off)
    pa, oa = tuple(c[rows].contiguous() for c in pg), _off(own)
    for mode in ("plain", "compensated"):
        total, em, pm = glv.glv_event_reduce(pg, og, mode=mode)
        ta, ea, ma = glv.glv_event_reduce(pa, oa, mode=mode)
        assert torch.equal(pm[pairs], ma)
        if mode == "plain":  # the compensated sums follow the events beside
            assert torch.equal(em[ev], ea)
        assert all(torch.equal(x[ev], y) for x, y in zip(total, ta))
        rank, bm = glv.glv_event_reduce_best_pair(pg, og, 91.2, mode=mode)
        ra, ba = glv.glv_event_reduce_best_pair(pa, oa, 91.2, mode=mode)
        assert torch.equal(rank[ev], ra) and torch.equal(bm[ev], ba)
    up = torch.from_numpy(g.standard_normal(int(po[-1]))).cuda().to(dtype)
    got = glv.glv_event_reduce_bwd(pg, og, grad_pair_m=up, tiling=(128, 64, 128, 512))
    want = glv.glv_event_reduce_bwd(pa, oa, grad_pair_m=up[pairs].contiguous(), tiling=(128, 64, 128, 512))
    assert all(torch.isfinite(c).all() for c in got)
    assert all(torch.equal(x[rows], y) for x, y in zip(got, want))
