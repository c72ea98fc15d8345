"""CPU: the division of the gain correction. The write pass forms fl(a / g), a = 0..255, as
q0 = a r, q = fmaf(fmaf(-q0, g, a), r, q0) with r = fl(1 / g), where every usable gain lies in
[2^-60, 2^60]; it must be the correctly rounded quotient (so that its rint, ties included, is the
definition's). fmaf is evaluated in double with the residual of the one inexact addition, which
settles the double rounding.
"""
import numpy as np
import pytest


def _fma32(a, b, c):
    """fl32(a b + c) for float32 arrays: the product is exact in double, the sum by TwoSum."""
    p, c = a.astype(np.float64) * b.astype(np.float64), c.astype(np.float64)
    s = p + c
    t = s - p
    err = (p - (s - t)) + (c - t)
    f = s.astype(np.float32)
    # s exactly between two floats, but the sum is not: take the side the residual lies on
    other = np.where(f.astype(np.float64) > s, np.nextafter(f, np.float32(-np.inf)),
                     np.nextafter(f, np.float32(np.inf)))
    mid = (f.astype(np.float64) + other.astype(np.float64)) / 2 == s
    up, down = np.maximum(f, other), np.minimum(f, other)
    return np.where(mid & (err > 0), up, np.where(mid & (err < 0), down, f))


@pytest.mark.parametrize("scale", [2.0 ** -60, 2.0 ** -7, 1.0, 2.0 ** 59])
def test_corrected_quotient_is_correctly_rounded(scale):
    rng = np.random.default_rng(11489)
    bits = np.concatenate([rng.integers(0, 1 << 23, 6000), np.arange(64), (1 << 23) - 1 - np.arange(64)])
    g = ((bits.astype(np.uint32) | np.uint32(127 << 23)).view(np.float32) * np.float32(scale))[:, None]
    a = np.arange(256, dtype=np.float32)[None, :]
    r = (1.0 / g.astype(np.float64)).astype(np.float32)   # double quotient to float: rounds as 1/g does
    q0 = a * r
    q = _fma32(_fma32(-q0, np.broadcast_to(g, q0.shape), np.broadcast_to(a, q0.shape)),
               np.broadcast_to(r, q0.shape), q0)
    assert np.array_equal(q, (a / g).astype(np.float32))
