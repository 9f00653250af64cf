"""The split of a float into three bf16 values and the six products that stand
for one (csrc/split.h), restated in numpy: the bounds that the header states,
and that the tolerance of the GPU tests sees a product that is missing."""
from __future__ import annotations

import numpy as np
import pytest

from gen import stream_rng

U = 2.0 ** -24
PRODUCTS = [(0, 2), (2, 0), (1, 1), (0, 1), (1, 0), (0, 0)]


def _bf16(v):
    """float32 values rounded to bf16, to nearest even"""
    u = v.astype(np.float32).view(np.uint32).astype(np.uint64)
    return ((u + 0x7fff + ((u >> 16) & 1)) & 0xffff0000).astype(np.uint32).view(np.float32)


def _split(v):
    h = _bf16(v)
    r = (v - h).astype(np.float32)
    m = _bf16(r)
    return h, m, _bf16((r - m).astype(np.float32))


def _product(a, b, left_out=None):
    A, B = _split(a), _split(b)
    return sum(A[i].astype(np.float64) * B[j] for i, j in PRODUCTS if (i, j) != left_out)


def test_split_is_exact():
    v = stream_rng(1, 1).standard_normal(200000).astype(np.float32)
    for e in (0, 100, -100, -109 + 24):
        s = (v * np.float32(2.0) ** e).astype(np.float32)
        s = s[np.abs(s) >= 2.0 ** -109]
        assert np.array_equal(sum(p.astype(np.float64) for p in _split(s)), s.astype(np.float64))


def test_product_bound():
    """The three products left out: at most 2^-24 of the product, 2^-26 as rms."""
    r = stream_rng(2, 1)
    a = (1 + r.random(2000000)).astype(np.float32)
    b = (1 + r.random(2000000)).astype(np.float32)
    rel = (_product(a, b) - a.astype(np.float64) * b) / (a.astype(np.float64) * b)
    assert np.max(np.abs(rel)) <= U
    assert np.sqrt(np.mean(rel ** 2)) <= U / 4


@pytest.mark.parametrize("left_out", PRODUCTS)
def test_missing_product_shows(left_out):
    """Sums of 64 products without one of the six are off by more than the
    eight units of 2^-24 (rms against rms) that the GPU tests allow."""
    r = stream_rng(3, 1)
    x = r.standard_normal((500, 64)).astype(np.float32)
    w = r.standard_normal((64, 30)).astype(np.float32)
    want = x.astype(np.float64) @ w.astype(np.float64)
    got = _product(x[:, :, None], w[None], left_out).sum(1)
    err = np.sqrt(np.mean((got - want) ** 2)) / np.sqrt(np.mean(want ** 2))
    full = _product(x[:, :, None], w[None]).sum(1)
    assert np.sqrt(np.mean((full - want) ** 2)) <= U / 2 * np.sqrt(np.mean(want ** 2))
    assert err > 16 * U
