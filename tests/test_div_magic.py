"""The quotient of the linear-site pass (div_rem with div_magic): one multiply
and one correction give the exact quotient and remainder of 32-bit operands."""
import numpy as np
import pytest


def _div_rem(n, d):
    m = np.uint64(0xFFFFFFFF if d <= 1 else (1 << 32) // d)
    n = n.astype(np.uint64)
    q = (n * m) >> np.uint64(32)
    r = n - q * np.uint64(d)
    fix = r >= d
    return q + fix, r - fix * np.uint64(d), r


@pytest.mark.parametrize("d", [1, 2, 3, 5, 7, 45, 63, 64, 65, 117, 150, 255, 256, 257, 1000, 4095,
                               4097, 65535, 65536, 65537, 2**31 - 1, 2**31, 2**32 - 1])
def test_div_rem_exact(d):
    g = np.random.default_rng(d)
    n = np.concatenate([g.integers(0, 2**32, 200000, dtype=np.uint64),
                        np.arange(0, 2000, dtype=np.uint64), 2**32 - 1 - np.arange(0, 2000, dtype=np.uint64)])
    k = g.integers(0, 2**32 // d + 1, 50000, dtype=np.uint64) * np.uint64(d)  # multiples and their neighbours
    n = np.concatenate([n, k, k + np.uint64(1), k - np.uint64(1)])
    n = n[n < 2**32]
    q, r, raw = _div_rem(n, d)
    assert (raw < 2 * d).all() and (raw < 2**32).all()
    assert (q == n // np.uint64(d)).all() and (r == n % np.uint64(d)).all()
