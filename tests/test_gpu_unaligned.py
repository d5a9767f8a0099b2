"""Columns at any element address (the rows of a block of odd length, a view
past the first element): bitwise what aligned copies of them give."""

import pytest
import torch

import oracle
import synth
from gpu_util import gpu

pytestmark = pytest.mark.gpu

glv = pytest.importorskip("paper_2312_02756_amd.glv")


def _rows(cols, pad):
    """Rows of one block whose row length puts them at differing offsets from 16 bytes."""
    n = cols[0].numel()
    block = torch.full((len(cols), n + pad), float("nan"), dtype=cols[0].dtype, device=cols[0].device)
    for r, c in zip(block, cols):
        r[pad:].copy_(c)
    return tuple(r[pad:] for r in block)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 6, 7, 127, 511, 514, 1025, 4099])
def test_rows_of_any_alignment(n, dtype):
    a, b = (gpu(x, dtype) for x in synth.pairs_generic(synth.rng(960 + n), n))
    cart = gpu(oracle.to_cartesian("PtEtaPhiM", [c.double().cpu().numpy() for c in a]), dtype)
    beta = tuple(0.2 * torch.tanh(c) for c in b[:3])
    mat = tuple(torch.sin(torch.arange(n, device=a[0].device, dtype=dtype) + k) for k in range(16))

    def calls(a, b, x, beta, m, up):
        out = []
        for mode in ("plain", "compensated"):
            out += [glv.glv_invariant_mass(a, b, mode=mode),
                    glv.glv_invariant_mass_histogram(a, b, 0.0, 300.0, 50, mode=mode)]
        out += [*sum(glv.glv_invariant_mass_bwd(a, b, up), ()), *sum(glv.glv_invariant_mass_comp_bwd(a, b, up), ()),
                *glv.glv_boost(x, beta), *sum(glv.glv_boost_bwd(x, beta, x), ()),
                *glv.glv_convert(a, "PtEtaPhiM", "PxPyPzE"), *glv.glv_convert(x, "PxPyPzE", "PtEtaPhiM"),
                *glv.glv_convert_bwd(a, x, "PtEtaPhiM", "PxPyPzE"),
                *glv.glv_lorentz_transform(x, m), *sum(glv.glv_lorentz_transform_bwd(x, m, x), ()),
                *glv.glv_rotate(x, m[:9]), *glv.glv_rotate_axis_angle(x, m[:4]),
                glv.glv_mass_histogram(up, -1.0, 1.0, 20)]
        return out

    up = torch.cos(a[0])
    want = calls(a, b, cart, beta, mat, up)
    for pad in (1, 2, 3):
        rows = _rows((*a, *b, *cart, *beta, *mat, up), pad)
        got = calls(rows[:4], rows[4:8], rows[8:12], rows[12:15], rows[15:31], rows[31])
        for k, (x, y) in enumerate(zip(got, want)):
            assert torch.equal(x.nan_to_num(7.0), y.nan_to_num(7.0)), (pad, k)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_unaligned_outputs_in_place(dtype):
    """Outputs over the unaligned inputs themselves, nothing written beside them."""
    n = 1027
    x = gpu(oracle.to_cartesian("PtEtaPhiM", synth.pairs_generic(synth.rng(961), n)[0]), dtype)
    beta = tuple(torch.full((1,), v, dtype=dtype, device=x[0].device) for v in (0.1, -0.2, 0.3))
    want = glv.glv_boost(x, beta)
    block = torch.full((4, n + 3), -7.0, dtype=dtype, device=x[0].device)
    rows = tuple(r[2:-1] for r in block)
    for r, c in zip(rows, x):
        r.copy_(c)
    glv.glv_boost(rows, beta, out=rows)
    assert all(torch.equal(r, w) for r, w in zip(rows, want))
    assert bool((block[:, :2] == -7.0).all()) and bool((block[:, -1] == -7.0).all())


@pytest.mark.parametrize("n", [(160 << 20) // 32 - 3, (160 << 20) // 32 + 5])
def test_cached_and_streamed_loads_agree(n):
    """A conversion of FP32 columns just under and over the size that streams: the first and last items bitwise
    those of a small call."""
    g = torch.Generator(device="cuda").manual_seed(962)
    x = tuple(torch.rand(n, device="cuda", generator=g) + 0.1 for _ in range(4))
    y = glv.glv_convert(x, "PtEtaPhiM", "PxPyPzE")
    for part in (slice(0, 1000), slice(n - 1001, n)):
        small = glv.glv_convert(tuple(c[part].clone() for c in x), "PtEtaPhiM", "PxPyPzE")
        assert all(torch.equal(c[part], s) for c, s in zip(y, small))


@pytest.mark.parametrize("n", [512, 511 * 512 * 2 + 1, 1024 * 1024 - 2, 1024 * 1024, 4096 * 1024 - 2, 4096 * 1024 + 3])
def test_fused_histogram_grids(n):
    """The sizes around which the fused histogram changes its number of workgroups: the counts of the stored masses."""
    a, b = (gpu(x, torch.float64) for x in synth.pairs_generic(synth.rng(963), n))
    got = glv.glv_invariant_mass_histogram(a, b, 0.0, 300.0, 1000)
    want = glv.glv_mass_histogram(glv.glv_invariant_mass(a, b), 0.0, 300.0, 1000)
    assert torch.equal(got, want) and int(got.sum()) == n
