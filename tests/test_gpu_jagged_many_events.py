"""Large events among 2^18 events and more, where the workgroups of the
large-event launches are given events instead of shares of the pairs."""

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import gpu
from paper_2312_02756_amd import _lib
from test_gpu_jagged import _off

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")


def _bwd_into(out, p, off, po, up):
    """glv_event_reduce_bwd of pair upstreams through the C ABI, without a tiling, into `out`."""
    cols = lambda c: _lib.P4(*[t.data_ptr() for t in c])  # noqa: E731
    dt = {torch.float64: _lib.GLV_F64, torch.float32: _lib.GLV_F32}[p[0].dtype]
    _lib.check("glv_event_reduce_bwd",
               _lib.load().glv_event_reduce_bwd(dt, _lib.GLV_PTETAPHIM, off.numel() - 1, off.data_ptr(), po.data_ptr(),
                                                cols(p), None, None, up.data_ptr(), cols(out), None,
                                                torch.cuda.current_stream().cuda_stream))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("ne", [(1 << 18) - 1, 1 << 18, (1 << 18) + 1, (3 << 20) + 77])
def test_large_events_first_and_last_of_many(ne, dtype):
    """Large events at the start, together in the middle and at the end of
    calls on either side of 2^18 events, and of more events than the threads
    of a launch look at in one go: every output of theirs is written, and
    bitwise as in a call of their own."""
    g = synth.rng(820)
    large = np.array([96, 41, 300, 130, 64, 97, 60, 1000, 49, 200], dtype=np.int64)
    at = np.array([0, 1, 2, 5, ne // 2, ne // 2 + 1, ne // 2 + 40, ne - 3, ne - 2, ne - 1])
    counts = g.integers(0, 4, ne)
    counts[at] = large
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    own = np.concatenate([[0], np.cumsum(large)]).astype(np.int64)
    po = oracle.pair_offsets(off)
    p, _ = synth.pairs_generic(g, int(off[-1]))
    rows = np.concatenate([np.arange(off[e], off[e + 1]) for e in at])
    pairs = np.concatenate([np.arange(po[e], po[e + 1]) for e in at])
    ev = torch.from_numpy(at).cuda()
    rows, pairs = torch.from_numpy(rows).cuda(), torch.from_numpy(pairs).cuda()
    pg, og = gpu(p, dtype), _off(off)
    pa, oa = tuple(c[rows].contiguous() for c in pg), _off(own)
    total, em, pm = glv.glv_event_reduce(pg, og)
    ta, ea, ma = glv.glv_event_reduce(pa, oa)
    assert torch.equal(pm[pairs], ma) and torch.equal(em[ev], ea)
    assert all(torch.equal(x[ev], y) for x, y in zip(total, ta))
    rank, bm = glv.glv_event_reduce_best_pair(pg, og, 91.2)
    ra, ba = glv.glv_event_reduce_best_pair(pa, oa, 91.2)
    assert torch.equal(rank[ev], ra) and torch.equal(bm[ev], ba)
    up = torch.from_numpy(g.standard_normal(int(po[-1]))).cuda().to(dtype)
    got = [torch.full_like(c, float("nan")) for c in pg]
    want = [torch.full_like(c, float("nan")) for c in pa]
    _bwd_into(got, pg, og, glv.glv_pair_offsets(og), up)
    _bwd_into(want, pa, oa, glv.glv_pair_offsets(oa), up[pairs].contiguous())
    assert all(torch.isfinite(c).all() for c in got)
    assert all(torch.equal(x[rows], y) for x, y in zip(got, want))
    assert all(torch.equal(x, y) for x, y in zip(got, glv.glv_event_reduce_bwd(pg, og, grad_pair_m=up)))
