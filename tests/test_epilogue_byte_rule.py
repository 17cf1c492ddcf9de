"""The product kernels' residue rule, checked on the host: an INT32 value x is given as
v = x + 2^31 modulo 2^32, the byte dot product of v with 2^(8 j) mod p brings it below
2^20, and the FP32 rule of the residue split gives the byte s + 128.  Evaluated for every
modulus on a window around 0, around half multiples of p over the whole range and at the
ends of the range, against the exact symmetric residue (p = 256: also for values that
wrapped around)."""
import numpy as np
import pytest

from oracle import core

BOUND = (1 << 17) * 127 * 127 + 3 * 127  # largest |x| for odd p
MODULI = [int(p) for p in core.constants(24)["p"]]


@pytest.mark.parametrize("p", MODULI)
def test_byte_rule(p):
    rng = np.random.default_rng(p)
    lim = (1 << 31) - 1 if p == 256 else BOUND
    half = rng.integers(-(lim // p), lim // p, 200000, dtype=np.int64) * p
    x = np.concatenate([np.arange(-100000, 100001, dtype=np.int64), np.array([-lim, lim]),
                        rng.integers(-lim, lim + 1, 500000, dtype=np.int64)]
                       + [np.clip(half + s * (p // 2) + d, -lim, lim) for s in (1, -1) for d in (-1, 0, 1)])
    v = (x + (1 << 31)) & 0xFFFFFFFF
    dot = sum(((v >> (8 * j)) & 0xFF) * pow(256, j, p) for j in range(4)) + 128 - pow(2, 31, p)
    assert np.abs(dot - 128).max() < 1 << 20
    ip = np.float32(1.0) / np.float32(p)
    rb = np.float32(0.5) - np.float32(128.0) * ip
    # fma: the product and the sum fit in 53 bits, one rounding to FP32
    q = np.floor((dot.astype(np.float64) * float(ip) + float(rb)).astype(np.float32))
    s = dot.astype(np.float64) - q.astype(np.float64) * p
    assert s.min() >= 0 and s.max() <= 255
    want = (x + p // 2) % p - p // 2 + 128  # [-floor(p/2), ceil(p/2) - 1] + 128
    assert np.array_equal(s.astype(np.int64), want)
