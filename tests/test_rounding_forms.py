"""The two forms of the stochastic rounding agree for every t they are used on: floor(t) + [k * 2^-24 < frac(t)] in fp32, and the
fixed-point one (csrc/device_math.hpp: sr_scale, sr_top, sr_pack), both restated here operation by operation.  A random word lies
on the edge between two codes once in 2^24 elements, so the words are put there."""
import numpy as np
import pytest

F = np.float32
MOST = F(127.0 * 2.0 ** 24)


def floating(t, k):
    f = np.floor(t)
    up = (k.astype(F) * F(2.0 ** -24)) < (t - f).astype(F)
    return np.clip(f.astype(np.int64) + up, -127, 127)


def fixed(t, k, one, lo, hi):
    """one: 1 where t < 0 (as fp32); lo, hi: bounds of -t * 2^24."""
    scaled = ((t + one).astype(F).astype(np.float64) * -2.0 ** 24 + one.astype(np.float64) * 2.0 ** 24).astype(F)   # the fma: exact in fp64
    c = np.floor(np.clip(scaled, lo, hi)).astype(np.int64)
    top = ((k ^ 0xFF000000) + c) & 0xFFFFFFFF
    byte = (~top & 0xFFFFFFFF) >> 24
    return byte - 256 * (byte > 127)


def values():
    rng = np.random.default_rng(5)
    mags = [2.0 ** -e * rng.uniform(1, 2, 400) for e in range(-6, 60)]
    whole = np.arange(0, 128, dtype=np.float64)
    edge = [127.0 + 2.0 ** -17, 127.0 - 2.0 ** -17, 0.5, 0.5 - 2.0 ** -26, 0.5 + 2.0 ** -24, 1 - 2.0 ** -24, 2.0 ** -24, 2.0 ** -25, 2.0 ** -26,
            3 * 2.0 ** -26, 2.0 ** -126, 2.0 ** -149, 0.0]
    v = np.concatenate([np.concatenate(mags), whole, whole + 0.5, edge]).astype(F)
    return v[v <= F(127.0 + 2.0 ** -17)]


def words(t):
    """Random words around the edge of each t, and the extremes."""
    frac = (t - np.floor(t)).astype(F).astype(np.float64) * 2.0 ** 24
    near = [np.floor(frac) + d for d in (-2, -1, 0, 1, 2)]
    ks = [np.clip(n, 0, 2 ** 24 - 1).astype(np.int64) for n in near]
    ks += [np.zeros(t.shape, np.int64), np.full(t.shape, 2 ** 24 - 1, np.int64), np.full(t.shape, 2 ** 23, np.int64)]
    return ks


@pytest.mark.parametrize("sign", [1, -1])
def test_fixed_point_rounding_is_the_floating_one(sign):
    t = (F(sign) * values()).astype(F)
    one = (np.ascontiguousarray(t).view(np.int32) >> 31 & 0x3F800000).view(F)
    zero = np.zeros_like(t)
    for k in words(t):
        ref = floating(t, k)
        assert np.array_equal(fixed(t, k, one, -MOST, MOST), ref)                       # sign taken from t
        if sign > 0:
            assert np.array_equal(fixed(t, k, zero, -MOST, F(0)), ref)                  # rectified, positive factor
            assert np.array_equal(fixed((-t).astype(F), k, zero, -MOST, F(0)), 0 * ref)   # rectified away
        else:
            assert np.array_equal(fixed(t, k, zero + F(1), F(0), MOST), ref)            # rectified, negative factor
            assert np.array_equal(fixed((-t).astype(F), k, zero + F(1), F(0), MOST), 0 * ref)
