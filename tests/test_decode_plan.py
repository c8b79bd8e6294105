"""The decode step's plan, on the host: what the workspace has to hold."""
import ctypes
import random

import pytest

from _host import compile_host, have_compiler

SOURCE = """
#include "hifa4_decode_plan.h"
using namespace hifa4;
// out: bps, packed, waves, runs, longest
extern "C" void plan(int batch, int hq, int hkv, int d, int nb, long tokens, long* out) {
  const DecodePlan p = plan_decode(batch, hq, hkv, d, nb, tokens);
  out[0] = p.bps; out[1] = p.packed; out[2] = p.waves; out[3] = p.runs; out[4] = p.longest;
}
extern "C" size_t room(int batch, int hq, int hkv, int d, int nb) {
  return decode_workspace_bytes(batch, hq, hkv, d, nb);
}
extern "C" size_t need(int batch, int hq, int d, long runs, long words, int packed) {
  size_t off[4];
  return decode_offsets(batch, hq, d, runs, words, packed, off);
}
"""


def load_plan(folder):
    lib = compile_host(SOURCE, folder)
    i, n = ctypes.c_int, ctypes.c_long
    lib.plan.argtypes, lib.plan.restype = [i, i, i, i, i, n, ctypes.POINTER(n)], None
    lib.room.argtypes, lib.room.restype = [i] * 5, ctypes.c_size_t
    lib.need.argtypes, lib.need.restype = [i, i, i, n, n, i], ctypes.c_size_t
    return lib


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    if not have_compiler():
        pytest.skip("g++ not available")
    return load_plan(tmp_path_factory.mktemp("plan"))


def plan(host, batch, hq, hkv, d, nb, tokens):
    out = (ctypes.c_long * 5)()
    host.plan(batch, hq, hkv, d, nb, tokens, out)
    return dict(zip(("bps", "packed", "waves", "runs", "longest"), out))


def test_workspace_holds_the_planned_and_the_grown_runs(host):
    rng = random.Random(7)
    for _ in range(20000):
        hkv = rng.choice([1, 2, 3, 4, 8, 12, 16, 64])
        hq, d = hkv * rng.randint(1, 8), rng.choice([64, 128, 256])
        batch, s = rng.choice([1, 2, 5, 8, 31, 64, 65, 256, 257, 1000]), int(2 ** rng.uniform(0, 19))
        nb = -(-s // 64)
        lens = [rng.randint(0, s) for _ in range(batch)]
        tokens = rng.choice([-1, 1, sum(lens)])
        p = plan(host, batch, hq, hkv, d, nb, tokens)
        room = host.room(batch, hq, hkv, d, nb)
        assert 1 <= p["bps"] <= 8
        words = max(p["runs"], p["longest"]) if p["packed"] else p["runs"]
        assert host.need(batch, hq, d, p["runs"], words, p["packed"]) <= room
        if p["packed"]:
            assert host.need(batch, hq, d, p["longest"], words, 0) <= room
            if tokens == sum(lens):          # the grid covers the lengths that it was planned for
                assert sum(-(-(-(-n // 64)) // p["bps"]) for n in lens) <= p["runs"]
            assert sum(-(-(-(-n // 64)) // 8) for n in lens) <= p["longest"]
        else:
            assert p["runs"] == batch * -(-nb // p["bps"])
