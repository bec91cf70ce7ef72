"""The FP32 convolutions' operand split on the CPU, over all 2^23 significands:
three BF16 pieces add up to the value exactly, rounded or cut off, and the
products of pieces that are left out (mid*lo, lo*mid, lo*lo) stay within 2^-24 of
the product, half an ulp, with rounded pieces."""

import numpy as np


def rounded(v):
    u = v.view(np.uint32).astype(np.uint64)
    return ((u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000).astype(np.uint32).view(np.float32)


def cut_off(v):
    return (v.view(np.uint32) & np.uint32(0xFFFF0000)).view(np.float32)


def pieces(x, f):
    hi = f(x)
    mid = f(x - hi)
    lo = f(x - hi - mid)
    assert np.array_equal(hi.astype(np.float64) + mid + lo, x.astype(np.float64))
    return hi, mid.astype(np.float64) / x, lo.astype(np.float64) / x


def widest(mid, lo):
    """Indices of the extreme (mid, lo) pairs: a bilinear form is largest there."""
    turns = np.linspace(0, 2 * np.pi, 33)
    return np.unique([np.argmax(mid * np.cos(t) + 512 * lo * np.sin(t)) for t in turns])


def test_pieces_are_exact_and_left_out_products_small():
    x = (np.arange(1 << 23, 1 << 24, dtype=np.int64) * 2.0 ** -23).astype(np.float32)
    hi, mid, lo = pieces(x, cut_off)
    assert (hi <= x).all() and (mid >= 0).all() and (lo >= 0).all()
    _, mid, lo = pieces(x, rounded)
    assert np.abs(mid).max() <= 2.0 ** -8 and np.abs(lo).max() <= 2.0 ** -17
    at = widest(mid, lo)
    left = np.abs(np.outer(mid[at], lo[at]) + np.outer(lo[at], mid[at]) + np.outer(lo[at], lo[at]))
    assert 2.0 ** -25 < left.max() <= 2.0 ** -24
