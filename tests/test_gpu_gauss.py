"""The kernels' Gaussian transform against the checker's, over every radius and every angle there is.

The transform takes 24 bits for the radius and 24 for the angle.  It is defined with a correctly rounded division and square
root; the kernels use one reciprocal (one reciprocal square root) and one residual correction, which rounds the same only because
the arguments lie in a narrow range.  That is a finite claim, so it is checked in full."""
import ctypes as C
from pathlib import Path

import numpy as np
import pytest

import oracle

ROOT = Path(__file__).resolve().parent.parent
WORDS = np.arange(1 << 24, dtype=np.uint32) << 8


def test_bulk_transform_is_the_pinned_one():
    rng = np.random.default_rng(5)
    xa, xb = rng.integers(0, 1 << 32, size=(2, 300), dtype=np.uint64).astype(np.uint32)
    zc, zs = oracle.gauss_pairs(xa, xb)
    assert [(float(c), float(s)) for c, s in zip(zc, zs)] == [oracle.gauss_pair(int(a), int(b)) for a, b in zip(xa, xb)]


@pytest.fixture(scope="module")
def transform():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    lib = C.CDLL(str(ROOT / "paper_2501_15129_amd" / "libes_microbench.so"))
    lib.es_gauss_words.argtypes = [C.c_void_p, C.c_void_p, C.c_uint32, C.c_void_p, C.c_void_p, C.c_void_p]

    def run(xa, xb):
        a, b = (torch.from_numpy(x.view(np.int32)).cuda() for x in (xa, xb))
        zc, zs = torch.empty(xa.size, device="cuda"), torch.empty(xa.size, device="cuda")
        assert lib.es_gauss_words(a.data_ptr(), b.data_ptr(), xa.size, zc.data_ptr(), zs.data_ptr(), None) == 0
        torch.cuda.synchronize()
        return zc.cpu().numpy(), zs.cpu().numpy()
    return run


def _same(got, want):
    for g, w in zip(got, want):
        differ = np.flatnonzero(g.view(np.uint32) != w.view(np.uint32))
        assert differ.size == 0, f"{differ.size} values differ, the first at {differ[0]}: {g[differ[0]]!r}, not {w[differ[0]]!r}"


@pytest.mark.gpu
def test_every_radius(transform):
    """Angle 0: the cosine is exactly 1 and the first value is the radius itself.  (The sine is 0, with its sign.)"""
    zero = np.zeros_like(WORDS)
    want = oracle.gauss_pairs(WORDS, zero)
    assert float(want[0].max()) > 5.7 and float(want[0].min()) == 0.0
    _same(transform(WORDS, zero), want)


@pytest.mark.gpu
def test_every_angle(transform):
    """With a radius that is a power of two the products are exact, so the values show the last bits of sine and cosine; the low
    eight bits of both words do not count."""
    radius = oracle.gauss_pairs(WORDS, np.zeros_like(WORDS))[0]
    exact = np.flatnonzero((radius.view(np.uint32) & 0x7FFFFF) == 0)
    exact = exact[radius[exact] > 0]
    assert exact.size > 0
    xa = np.full_like(WORDS, WORDS[exact[0]])
    _same(transform(xa, WORDS), oracle.gauss_pairs(xa, WORDS))
    _same(transform(xa | 0xFF, WORDS | 0xA5), oracle.gauss_pairs(xa, WORDS))
