"""The three-term bf16 split of the chunk kernels, restated on the CPU over
every fp32 significand: it is exact, and the products that the kernels leave out
(mid x low, low x mid, low x low) are at most 2^-24 of the product."""
import numpy as np


def bf16(x):
    """Rounded to the nearest bf16 (ties to even), as fp32."""
    u = x.view(np.uint32).astype(np.uint64)
    u = (u + 0x7FFF + ((u >> 16) & 1)) & 0xFFFF0000
    return u.astype(np.uint32).view(np.float32)


def split(x):
    h = bf16(x)
    r = x - h
    m = bf16(r)
    return h, m, bf16(r - m)


def test_split_of_every_significand():
    x = (np.arange(1 << 23, dtype=np.uint32) | np.uint32(127 << 23)).view(np.float32)
    h, m, low = split(x)
    x64, h, m, low = (a.astype(np.float64) for a in (x, h, m, low))
    assert np.array_equal(h + m + low, x64)
    mid, last = np.max(np.abs(m) / x64), np.max(np.abs(low) / x64)
    assert mid <= 2.0 ** -8 and last <= 2.0 ** -17
    assert 2 * mid * last + last * last <= 1.01 * 2.0 ** -24


def test_split_holds_across_the_exponents_in_use():
    """From 2^59 (larger operands are formed in fp32) down to where the lowest
    term leaves fp32's normal range."""
    r = np.random.default_rng(1)
    s = r.integers(0, 1 << 23, 4096, dtype=np.uint32)
    for e in range(127 - 102, 127 + 59):
        x = (s | np.uint32(e << 23)).view(np.float32)
        assert np.array_equal(sum(a.astype(np.float64) for a in split(x)), x.astype(np.float64)), e
