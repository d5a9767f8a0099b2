"""Tilings on the host (no GPU needed): what a call is launched with, and what
it refuses, through the C ABI.  Pointers are fake addresses; no call below
reaches a launch."""

import ctypes
import json

import pytest
import torch

from paper_2312_02756_amd import _lib, glv

OK, NULL, SIZE, DTYPE, COORDS, MODE, TILING = 0, 1, 2, 3, 4, 5, 9
DEFAULT_BWD = (128, 64, 128, 512)


@pytest.fixture(scope="module")
def lib():
    return _lib.load()


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("GLV_AUTOTUNE_CACHE", str(path))
    glv.glv_autotune_forget()
    yield path
    glv.glv_autotune_forget()


def _tune(path, tiling, **kw):
    """Makes `tiling` the tuned choice of this process."""
    key = glv.glv_autotune_key(None, **kw)
    path.write_text(json.dumps({"format": "glv-autotune-1", "entries": [{"key": key, "tiling": list(tiling)}]}))
    assert glv.glv_autotune_lookup(None, **kw) == (tiling, True)


def test_call_tiling_validation(lib):
    t = _lib.glv_tiling()
    f, out = lib.glv_call_tiling, ctypes.byref(t)
    assert f(3, 1, 0, 0, 10, 10, out) == DTYPE
    assert f(2, 4, 0, 0, 10, 10, out) == COORDS
    assert f(2, 0, 1, 0, 10, 10, out) == MODE
    assert f(2, 0, 1, 1, 10, 10, out) == OK      # the reverse mode has one mode
    assert f(2, 1, 0, 0, -1, 10, out) == SIZE
    assert f(2, 1, 0, 0, 10, -2, out) == SIZE
    assert f(2, 1, 0, 0, 10, 10, None) == NULL


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_untuned_sizes_are_valid_and_follow_the_events(lib, dtype):
    """Every choice fits the LDS, and few events get small tiles."""
    glv.glv_autotune_forget()
    code, es = (2, 8) if dtype == torch.float64 else (1, 4)
    for ne in (0, 1, 8192, 8193, 32768, 131072, 131073, 1 << 19, (1 << 19) + 1, 1 << 21):
        for mean in (None, 0, 1, 10, 44, 46, 89, 91, 149, 151, 349, 351, 1249, 1251, 100000):
            n_pairs = None if mean is None else mean * ne
            for mode in ("plain", "compensated"):
                t = _lib.glv_tiling(*glv.glv_call_tiling(ne, n_pairs, dtype, "PtEtaPhiM", mode))
                # no events: the tiling is checked and nothing is launched
                assert lib.glv_event_reduce(code, 1, mode == "compensated", 0, None, None, None, None, None, None, None,
                                            ctypes.byref(t), None) == OK
            block, epb, cap, q = glv.glv_call_tiling(ne, n_pairs, dtype, backward=True)
            assert block in (64, 128, 256, 512) and 1 <= epb <= 64 and 64 <= cap <= block and q % 64 == 0 and q <= 4096
            assert cap * (4 * es + 2) + (q + 2) * es + epb * (4.5 * es + 32) + 64 <= 65536
            assert epb <= (4 if ne <= 8192 else 64)


def test_pairs_decide_the_reverse_mode_where_they_are_known(cache):
    assert glv.glv_call_tiling(500000, 500000 * 98, torch.float32, backward=True) == (256, 64, 256, 4096)
    assert glv.glv_call_tiling(60000, 60000 * 325, torch.float64, backward=True) == (256, 16, 256, 2048)
    assert glv.glv_call_tiling(500000, 500000 * 32, torch.float32, backward=True) == glv.glv_call_tiling(
        500000, None, torch.float32, backward=True)
    assert glv.glv_call_tiling(500000, 0, torch.float32, backward=True) == DEFAULT_BWD  # no pair upstreams


def test_reverse_mode_of_many_fp64_events(cache):
    """The number of events alone does not take the room for pairs away: only
    small events, which do not need it, have less of it."""
    for ne in (500000, 600000, 1 << 21):
        assert glv.glv_call_tiling(ne, None, backward=True) == (128, 32, 128, 768)
        assert glv.glv_call_tiling(ne, 48 * ne, backward=True) == (128, 32, 128, 768)
        assert glv.glv_call_tiling(ne, 98 * ne, backward=True) == (256, 64, 256, 2048)
    assert glv.glv_call_tiling(500000, 32 * 500000, backward=True) == (128, 32, 128, 768)
    assert glv.glv_call_tiling(600000, 32 * 600000, backward=True) == DEFAULT_BWD


@pytest.mark.parametrize("tiling", [DEFAULT_BWD, (64, 16, 64, 256)])
def test_a_tuned_choice_is_taken_whatever_it_is(cache, tiling):
    """Also one that equals the built-in default."""
    _tune(cache, tiling, backward=True)
    for n_pairs in (None, 60000 * 325):
        assert glv.glv_call_tiling(60000, n_pairs, backward=True) == tiling
    assert glv.glv_call_tiling(60000, 60000 * 325, torch.float32, backward=True) != tiling  # another key


@pytest.mark.parametrize("backward", [False, True])
def test_a_lookup_that_finds_nothing_leaves_the_call_untuned(cache, backward):
    """It reports the default, as ever, and the call takes what an untuned one
    does."""
    kw = dict(dtype=torch.float64, backward=backward)
    untuned = glv.glv_call_tiling(1000, 98000, **kw)
    current = glv.glv_current_tiling_bwd if backward else glv.glv_current_tiling
    default = current(torch.float64)
    assert untuned != default and untuned[1] == 4
    assert glv.glv_autotune_lookup(None, **kw) == (default, False)
    assert glv.glv_call_tiling(1000, 98000, **kw) == untuned
    _tune(cache, (64, 16, 64, 128), **kw)
    assert glv.glv_call_tiling(1000, 98000, **kw) == (64, 16, 64, 128)
    cache.unlink()
    glv.glv_autotune_forget()
    _tune(cache, (64, 16, 64, 128), **kw)
    cache.write_text(json.dumps({"format": "glv-autotune-1", "entries": []}))
    assert glv.glv_autotune_lookup(None, **dict(kw, dtype=torch.float32)) != ((64, 16, 64, 128), True)
    assert glv.glv_call_tiling(1000, 98000, **kw) == (64, 16, 64, 128)  # another key's miss changes nothing


GiB = 1 << 30


def _cols(base):
    return _lib.P4(*[base + i * GiB for i in range(4)])


@pytest.mark.parametrize("ne", [1, 10, 8192, 32768, 131072, 1 << 20])
def test_partly_given_tilings_are_refused_at_any_number_of_events(lib, ne):
    """A field left 0 beside given ones is the current choice whatever the
    number of events, so that a tiling that asks for too much LDS with it is
    refused for few events as for many."""
    glv.glv_autotune_forget()
    off, po, p, t, em, pm = 16 * GiB, 32 * GiB, _cols(100 * GiB), _cols(140 * GiB), 180 * GiB, 190 * GiB
    for bad in ((512, 0, 140, 448), (512, 0, 128, 512), (256, 0, 300, 896)):
        b = ctypes.byref(_lib.glv_tiling(*bad))
        assert lib.glv_event_reduce(2, 1, 0, ne, off, po, p, t, em, pm, None, b, None) == TILING, bad
    for bad in ((512, 0, 208, 64), (256, 0, 464, 64)):
        b = ctypes.byref(_lib.glv_tiling(*bad))
        assert lib.glv_event_reduce_best_pair(2, 1, 0, ne, off, po, p, 91.0, 140 * GiB, em, None, b, None) == TILING, bad


@pytest.mark.parametrize("mode", ["plain", "compensated"])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
def test_tiles_of_the_forward_stay_small_up_to_393216_events(cache, dtype, mode):
    """Where pairs are evaluated; without them, and in the reverse mode, up to 131,072."""
    for n_pairs in (None, 1 << 22):
        tile = lambda ne: glv.glv_call_tiling(ne, n_pairs, dtype, mode=mode)[1]  # noqa: E731
        assert tile(32769) == tile(131073) == tile(393216) == 16
        assert tile(393217) == tile(1 << 22) > 16
    assert glv.glv_call_tiling(131073, 0, dtype, mode=mode)[1] > 16
    assert glv.glv_call_tiling(131073, None, dtype, backward=True)[1] > 16
