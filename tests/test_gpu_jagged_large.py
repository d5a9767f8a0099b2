"""Events of many particles (the large-event launches of the jagged reduction
and its reverse mode) against the CPU oracle, at the edges of their blocks,
chunks and tiles: 32 particles per backward block, 64 partners per batch, 128
particles summed by quads, 256 and 512 staged, and beyond."""

import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_util import gpu, host, widened
from test_gpu_jagged import _check_bwd, _check_forward, _off
from tolerances import U64, worst

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")

EDGES = [31, 32, 33, 34, 47, 48, 49, 50, 63, 64, 65, 66, 95, 96, 97, 127, 128, 129, 191, 192, 193, 255, 256, 257]
WIDE = [511, 512, 513, 770, 1025]


def _csr(counts, start=0):
    off = np.zeros(len(counts) + 1, dtype=np.int64)
    off[1:] = np.cumsum(counts)
    return off + start


def _mixed(sizes, seed):
    """The sizes in random order between runs of small events."""
    g = synth.rng(seed)
    counts = []
    for n in g.permutation(sizes):
        counts += [int(n)] + [int(c) for c in g.integers(0, 12, int(g.integers(0, 4)))]
    return np.array(counts, dtype=np.int64)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("mode", ["plain", "compensated"])
def test_large_events_forward_and_best(mode, dtype):
    """Every mass and total against the oracle; the fused best pair bitwise the
    one selected from the stored masses.  FP64 event masses of the compensated
    mode against the binary128 sums instead of the binary64 ones, which add up
    to 524,800 terms one after the other (off by 111 u on 513 particles)."""
    off = _csr(_mixed(EDGES + WIDE, 801))
    p, _ = synth.pairs_generic(synth.rng(802), int(off[-1]))
    pg, og = gpu(p, dtype), _off(off)
    total, em, pm = glv.glv_event_reduce(pg, og, mode=mode)
    if mode == "compensated" and dtype == torch.float64:
        em_q = oracle.event_reduce_q("PtEtaPhiM", off, p)[1]
        # events of one particle: its own mass, which the plain sums of binary128 give to less than u
        r, i = worst(np.abs(host(em) - em_q), 64 * U64 * em_q + 1e-300)
        assert r <= 1.0, ("event_m", i, host(em)[i], em_q[i])
        em = oracle.event_reduce("PtEtaPhiM", off, p, mode=oracle.ACCURATE)[1]
        em = torch.from_numpy(em)
    _check_forward(off, p, dtype, "PtEtaPhiM", mode, total, em, pm, f"large {mode} {dtype}")
    rank, bm = glv.glv_event_reduce_best_pair(pg, og, 91.2, mode=mode)
    want_r, want_m = glv.glv_event_best_pair(glv.glv_pair_offsets(og), pm, 91.2)
    assert np.array_equal(host(rank), host(want_r))
    assert np.array_equal(host(bm), host(want_m), equal_nan=True)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("coords", ["PtEtaPhiM", "PxPyPzE"])
def test_large_events_backward(coords, dtype):
    off = _csr(_mixed(EDGES + [385, 520], 803))
    g = synth.rng(804)
    p, _ = synth.pairs_generic(g, int(off[-1]))
    if coords == "PxPyPzE":
        p = oracle.to_cartesian("PtEtaPhiM", p)
    ne = off.size - 1
    gt = synth.upstream(g, ne, 4)
    gem = g.standard_normal(ne)
    gpr = g.standard_normal(int(oracle.pair_offsets(off)[-1]))
    wp = widened(p, dtype)
    want = oracle.event_reduce_vjp(coords, off, wp, widened(gt, dtype), widened([gem], dtype)[0],
                                   widened([gpr], dtype)[0])
    pg, og = gpu(p, dtype), _off(off)
    kw = dict(grad_total=gpu(gt, dtype), grad_event_m=gpu([gem], dtype)[0], grad_pair_m=gpu([gpr], dtype)[0],
              coords=coords)
    total = glv.glv_event_reduce(pg, og, coords=coords)[0]
    for tot in (None, total):
        got = glv.glv_event_reduce_bwd(pg, og, total=tot, **kw)
        _check_bwd(off, wp, dtype, coords, [host(c).astype(np.float64) for c in got], want, f"totals {tot is not None}")


@pytest.mark.parametrize("large_first", [True, False])
def test_large_events_far_from_their_expected_place(large_first):
    """40 large events before or after 150,000 tiny ones: the shares of pairs
    begin far from where equal events would put them, so that they are
    searched for.  Every large event bitwise as in a call of its own, with
    particles and offsets that do not start at 0."""
    g = synth.rng(805)
    large = np.array(g.integers(40, 400, 40), dtype=np.int64)
    small = np.array(g.integers(0, 3, 150000), dtype=np.int64)
    counts = np.concatenate([large, small] if large_first else [small, large])
    off = _csr(counts, 7)
    n = int(off[-1])
    p, _ = synth.pairs_generic(g, n)
    e0 = 0 if large_first else small.size
    lo, hi = int(off[e0]), int(off[e0 + large.size])
    po = oracle.pair_offsets(off)
    q0, q1 = int(po[e0]), int(po[e0 + large.size])
    alone = _off(_csr(large))
    for dtype in (torch.float64, torch.float32):
        pg, og = gpu(p, dtype), _off(off)
        pa = tuple(c[lo:hi].clone() for c in pg)
        total, em, pm = glv.glv_event_reduce(pg, og)
        ta, ea, ma = glv.glv_event_reduce(pa, alone)
        assert torch.equal(pm[q0:q1], ma) and torch.equal(em[e0:e0 + large.size], ea)
        assert all(torch.equal(a[e0:e0 + large.size], b) for a, b in zip(total, ta))
        up = torch.from_numpy(g.standard_normal(int(po[-1]))).to(og.device).to(dtype)
        gp = glv.glv_event_reduce_bwd(pg, og, grad_pair_m=up)
        ga = glv.glv_event_reduce_bwd(pa, alone, grad_pair_m=up[q0:q1].clone())
        assert all(torch.equal(a[lo:hi], b) for a, b in zip(gp, ga))
        rank, bm = glv.glv_event_reduce_best_pair(pg, og, 91.2)
        ra, ba = glv.glv_event_reduce_best_pair(pa, alone, 91.2)
        assert torch.equal(rank[e0:e0 + large.size], ra) and torch.equal(bm[e0:e0 + large.size], ba)


@pytest.mark.parametrize("ne", [2047, 2048, 2049, 4 * 2048 + 1, 65535, 65536, 65537, 2048 * 33])
def test_pair_offsets_at_tile_and_launch_edges(ne):
    """Tiles of 2,048 events; one launch up to 65,536 events, three beyond."""
    off = _csr(synth.rng(806 + ne).integers(0, 20, ne))
    assert np.array_equal(host(glv.glv_pair_offsets(_off(off))), oracle.pair_offsets(off))


@pytest.mark.parametrize("mode,dtype,n", [("plain", torch.float64, 24), ("plain", torch.float32, 24),
                                          ("compensated", torch.float64, 18), ("compensated", torch.float32, 22)])
def test_line_between_the_launches(mode, dtype, n):
    """Mean pairs just below and above the number from which the second launch
    takes all but the smallest events."""
    for size in (n, n + 1):
        off = _csr([size] * 40 + [1, 0, size - 1])
        p, _ = synth.pairs_generic(synth.rng(808 + size), int(off[-1]))
        pg, og = gpu(p, dtype), _off(off)
        total, em, pm = glv.glv_event_reduce(pg, og, mode=mode)
        _check_forward(off, p, dtype, "PtEtaPhiM", mode, total, em, pm, f"line {size} {mode} {dtype}")


@pytest.mark.parametrize("tiling", [(0, 0, 0, 0), (64, 1, 64, 64), (64, 64, 4000, 4096), (256, 64, 950, 4096),
                                    (512, 64, 447, 4096), (512, 1, 500, 128), (128, 7, 100, 192)])
@pytest.mark.parametrize("sizes", [[48, 2, 47, 0, 1, 48] + [0] * 9, [9] * 130, [2] * 300, [30, 3] * 50])
def test_fp32_rounds_of_any_tiling(tiling, sizes):
    """FP32 plain masses staged in rounds, up to the tilings whose particles
    leave the least LDS for them: those of the oracle
    and bitwise those of another tiling."""
    off = _csr(sizes, 3)
    p, _ = synth.pairs_generic(synth.rng(809), int(off[-1]))
    pg, og = gpu(p, torch.float32), _off(off)
    total, em, pm = glv.glv_event_reduce(pg, og, tiling=tiling)
    _check_forward(off, p, torch.float32, "PtEtaPhiM", "plain", total, em, pm, f"rounds {tiling}")
    ref = glv.glv_event_reduce(pg, og, tiling=(256, 16, 128, 256))
    assert torch.equal(pm, ref[2]) and torch.equal(em, ref[1])
    assert all(torch.equal(a, b) for a, b in zip(total, ref[0]))


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("ne,sizes", [(131072, (2, 5)), (131073, (2, 5)), (524288, (1, 3)), (524289, (1, 3)),
                                      (700, (39, 40, 41, 45, 46, 47)), (700, (54, 55, 56, 57, 4))])
def test_reverse_mode_chunks_without_a_tiling(ne, sizes, dtype):
    """Event counts and event sizes around which the chunks of the reverse mode
    change, through the binding and by the C ABI's own choice: small events
    bitwise as with a given tiling, larger ones (whose sums follow the launch
    they are done in) the oracle's gradients."""
    g = synth.rng(810 + ne)
    off = _csr(g.choice(sizes, ne))
    p, _ = synth.pairs_generic(g, int(off[-1]))
    gpr = g.standard_normal(int(oracle.pair_offsets(off)[-1]))
    gem, gt = g.standard_normal(ne), synth.upstream(g, ne, 4)
    pg, og = gpu(p, dtype), _off(off)
    kw = dict(grad_total=gpu(gt, dtype), grad_event_m=gpu([gem], dtype)[0], grad_pair_m=gpu([gpr], dtype)[0])
    got = [glv.glv_event_reduce_bwd(pg, og, tiling=t, **kw) for t in (None, (0, 0, 0, 0), (64, 16, 64, 512))]
    if max(sizes) < 10:
        assert all(torch.equal(a, b) for o in got[:2] for a, b in zip(o, got[2]))
        return
    wp = widened(p, dtype)
    want = oracle.event_reduce_vjp("PtEtaPhiM", off, wp, widened(gt, dtype), widened([gem], dtype)[0],
                                   widened([gpr], dtype)[0])
    for o in got:
        _check_bwd(off, wp, dtype, "PtEtaPhiM", [host(c).astype(np.float64) for c in o], want, f"chunks {ne} {sizes}")
