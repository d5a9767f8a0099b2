"""Plain pair masses are the same whichever launch of the jagged reduction an
event is done in.  The two take different roots in FP32 (sqrtf; the hardware's
reciprocal root and one residual step, valid from 2^-102 on), so the pairs' m^2
here cover every exponent, the values around that line and its guard at 2^-96,
zero, infinity and NaN, and a binade pair densely."""

import numpy as np
import pytest
import torch

import synth
from test_gpu_jagged import _off

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")

N = 20  # particles per event: 190 pairs, for a mean of which the first launch does them; for one of 1,000 the second


def _cartesian(scale, g, dtype):
    """(px, py, pz, E) of events of N particles whose components are of the order of scale[e]."""
    s = np.repeat(scale, N)
    e = s * g.uniform(0.5, 1.0, s.size)
    p = [e * g.uniform(-1.2, 1.2, s.size) * (g.random(s.size) < 0.5) for _ in range(3)]
    with np.errstate(over="ignore", under="ignore"):
        return tuple(torch.from_numpy(c.astype(np.float32 if dtype == torch.float32 else np.float64)) for c in (*p, e))


def _bits(x):
    return x.view(torch.int32 if x.dtype == torch.float32 else torch.int64)


def _both_launches(cols, ne):
    """Pair masses of the events alone (first launch) and with large events behind them (second launch)."""
    alone = np.arange(ne + 1, dtype=np.int64) * N
    large = 200
    extra = (ne * 810) // (large * (large - 1) // 2 - 1000) + 1  # so that the mean passes 1,000 pairs
    counts = np.concatenate([np.full(ne, N), np.full(extra, large)])
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int64)
    pairs = counts * (counts - 1) // 2
    assert pairs[:ne].mean() == 190 and pairs.mean() >= 1000
    pad = [torch.ones(extra * large, dtype=c.dtype) * (1.0 if k == 3 else 0.1) for k, c in enumerate(cols)]
    first = glv.glv_event_reduce(tuple(c.cuda() for c in cols), _off(alone), coords="PxPyPzE")
    second = glv.glv_event_reduce(tuple(torch.cat([c, d]).cuda() for c, d in zip(cols, pad)), _off(off),
                                  coords="PxPyPzE")
    nq = ne * (N * (N - 1) // 2)
    return (first[2], second[2][:nq]), [(a, b[:ne]) for a, b in zip((*first[0], first[1]), (*second[0], second[1]))]


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_masses_of_every_exponent(dtype):
    g = synth.rng(830)
    lo, hi = (-76, 66) if dtype == torch.float32 else (-540, 515)
    exponents = np.repeat(np.arange(lo, hi), 40)
    if dtype == torch.float32:  # m^2 around 2^-102 and 2^-96, and at the largest floats
        exponents = np.concatenate([exponents, np.repeat([-52, -51, -50, -49, -48, -47, 62, 63], 400)])
    cols = _cartesian(2.0 ** exponents, g, dtype)
    special = g.permutation(exponents.size)[:200] * N  # the first particle of some events
    for k, v in enumerate((0.0, np.inf, -np.inf, np.nan)):
        for c in cols:
            c[torch.from_numpy(special[k * 50:(k + 1) * 50])] = v
    (a, b), rest = _both_launches(cols, exponents.size)
    assert torch.equal(_bits(a), _bits(b))
    for x, y in rest:
        assert torch.equal(_bits(x), _bits(y))
    m = a[torch.isfinite(a) & (a != 0)].abs().double()
    span = (-74, 63) if dtype == torch.float32 else (-537, 511)
    assert float(m.log2().min()) < span[0] + 4 and float(m.log2().max()) > span[1]  # the range was met


def test_fp32_masses_of_a_binade_pair():
    """9.5 million m^2 between 1/4 and 4."""
    g = synth.rng(831)
    ne = 50000
    e = g.uniform(0.25, 1.0, ne * N)
    cols = tuple(torch.from_numpy(c.astype(np.float32)) for c in (e * g.uniform(-0.2, 0.2, e.size), 0 * e, 0 * e, e))
    (a, b), _ = _both_launches(cols, ne)
    assert torch.equal(a, b)
