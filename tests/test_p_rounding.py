"""The attention kernels' packed-fp16 rounding of P and the multiplicative base,
restated in numpy and compared with the HIF4 definition for every fp16 input."""
import numpy as np
import pytest

E6M2 = (1.0 + (np.arange(256) & 3) / 4.0) * np.exp2((np.arange(256) >> 2) - 31.0)
R16 = (32800.0, 26224.0, 21856.0, 18736.0)         # 2^15 / (1 + m/4), taken just above


def test_base_by_product_is_the_smallest_covering_base():
    a = np.arange(1, 0x7C00, dtype=np.uint16).view(np.float16)
    y = (a.astype(np.float32) * np.float32(float.fromhex("0x1.249236p-1"))).astype(np.float32)
    b = ((y.view(np.uint32) + np.uint32(0x1FFFFF)) & np.uint32(0xFFE00000)).view(np.float32)
    assert np.array_equal(b.astype(np.float64), E6M2[np.searchsorted(1.75 * E6M2, a.astype(np.float64))])


@pytest.mark.parametrize("m", range(4))
def test_floor_then_fma_is_round_half_away(m):
    p_all = np.arange(0, 0x3C01, dtype=np.uint16).view(np.float16).astype(np.float64)
    assert float(np.float16(R16[m])) == R16[m]
    for e in range(-25, 0):                         # the bases a block maximum in (0, 1] can have
        b = (1 + m / 4) * 2.0 ** e
        assert float(np.float16(2.0 ** (-17 - e))) == 2.0 ** (-17 - e)
        for sh in range(3):
            step = b / 4 * 2.0 ** -sh
            p = p_all[p_all <= 7 * step]
            w = np.floor(p * 2.0 ** (7 - e))        # the truncating multiply, in units of 2^-24
            assert w.max() < 1024
            c = 1.5 * 2.0 ** (6 - sh)
            o = (w * 2.0 ** -24 * R16[m] + c).astype(np.float16).astype(np.float64) - c     # exact before the rounding
            assert np.array_equal(o * 16 * 2 ** sh, np.floor(p / step + 0.5))
