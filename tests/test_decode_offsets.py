"""The decode kernel's copies of a 64-key block clamp each row's byte offset to
the last key they may read.  Emulated for every row of first, middle and last
blocks, with K^ caches on both sides of 4 GiB: row r reads key min(r, last)."""
import ctypes

import numpy as np
import pytest

from _host import compile_host, have_compiler

SOURCE = """
#include "hifa4_decode_plan.h"
extern "C" uint32_t last_key_offset(int left, uint32_t row_bytes) { return hifa4::last_key_offset(left, row_bytes); }
"""


@pytest.fixture(scope="module")
def last_key_offset(tmp_path_factory):
    if not have_compiler():
        pytest.skip("g++ not available")
    f = compile_host(SOURCE, tmp_path_factory.mktemp("offsets")).last_key_offset
    f.restype, f.argtypes = ctypes.c_uint32, [ctypes.c_int, ctypes.c_uint32]
    return f


@pytest.mark.parametrize("length,hkv,d", [
    (1, 1, 64), (64, 8, 128), (100, 12, 256), (32768, 8, 128),
    (1048577, 32, 256), (2097200, 32, 128), (8388700, 8, 128),     # the end lies past 2^32 bytes of codes
    ((1 << 31) - 1, 1, 64),                                         # most tokens of one head
])
def test_every_row_reads_its_key(last_key_offset, length, hkv, d):
    row = hkv * d // 2
    last_block = (length - 1) // 64
    for block in sorted({0, 1, last_block // 2, last_block - 1, last_block} & set(range(last_block + 1))):
        left = length - 64 * block
        want = np.minimum(np.arange(64), left - 1)
        limit = last_key_offset(left, row)
        got = np.minimum(np.arange(64, dtype=np.uint64) * row, limit)
        assert np.array_equal(got, want * row), (block, limit)
