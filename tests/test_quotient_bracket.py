"""The K smoothing quotient's bracket (two fp32 products with the reciprocal two
ulps down and up): where both round to the same fp16, so does the exact k/s."""
import numpy as np

from oracle.smooth import _round_quotient_fp16


def _bracket(k, s):
    r = (np.float32(1.0) / s).astype(np.float32)
    lo = (r.view(np.uint32) - np.uint32(2)).view(np.float32)
    hi = (r.view(np.uint32) + np.uint32(2)).view(np.float32)
    k32 = k.astype(np.float32)
    with np.errstate(over="ignore"):
        return (k32 * lo).astype(np.float16), (k32 * hi).astype(np.float16)


def test_equal_ends_give_the_rounded_quotient():
    rng = np.random.default_rng(5)
    n = 1 << 20
    s = np.exp(rng.uniform(-6, 6, 2 * n)).astype(np.float32)
    k = np.empty(2 * n, np.float16)
    k[:n] = (rng.standard_normal(n) * rng.choice([1e-6, 1e-3, 1.0, 100.0], n)).astype(np.float16)
    mid = rng.integers(1, 0x7400, n).astype(np.uint16).view(np.float16).astype(np.float64)   # quotients near midpoints
    up = np.nextafter(mid.astype(np.float16), np.float16(np.inf)).astype(np.float64)
    with np.errstate(over="ignore"):
        k[n:] = ((mid + up) / 2 * s[n:]).astype(np.float16)
    k[n:] *= rng.choice([-1, 1], n).astype(np.float16)
    ok = np.isfinite(k)
    k, s = k[ok], s[ok]
    a, b = _bracket(k, s)
    same = a == b
    want = _round_quotient_fp16(k, s)
    assert np.array_equal(a[same], want[same])
    assert np.count_nonzero(~same[:n]) < n / 400          # the exact division stays rare on ordinary values
