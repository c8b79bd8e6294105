"""The decode kernel's copies into LDS set M0 in the statement that issues
them, and the compiler keeps no value of its own there: in the compiled decode
translation unit every instruction that names M0 is such a write, immediately
followed by its scalar-base load."""
import os
import re
import subprocess

import pytest

from test_m0_guard import ROOT, _hipcc


@pytest.mark.skipif(_hipcc() is None, reason="hipcc not available")
def test_m0_is_only_the_block_copies(tmp_path):
    out = tmp_path / "decode.s"
    cmd = [_hipcc(), "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "--cuda-device-only", "-S", "-x", "hip",
           os.path.join(ROOT, "paper_2607_04302_amd", "csrc", "hifa4_decode.hip"), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True, timeout=600)
    lines = [l.strip() for l in out.read_text().splitlines()]
    code = [l for l in lines if l and not l.startswith((";", ".", "_")) and not l.endswith(":")]
    writes = 0
    for i, l in enumerate(code):
        if not re.search(r"\bm0\b", l):
            continue
        assert l.startswith("s_mov_b32 m0,"), f"M0 used outside the copies: {l}"
        nxt = code[i + 1] if i + 1 < len(code) else ""
        assert nxt.startswith("global_load_lds_dword") and ", s[" in nxt, (l, nxt)
        writes += 1
    assert writes > 0, "no copies into LDS found"
