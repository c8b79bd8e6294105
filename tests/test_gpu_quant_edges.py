"""The canonical quantizers and the calibration pass at the sizes where their
work split can go wrong, against the oracle: bit-exact codes, metadata and gate
statistics, scales within one fp32 ulp."""
import numpy as np
import pytest

from oracle import attention as oatt
from oracle import smooth as osmooth

from _gpu_util import to_gpu, to_np

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def h():
    import paper_2607_04302_amd as mod
    mod.load_library()
    return mod


def _draw(rng, *shape):
    x = (rng.standard_normal(shape) * 4).astype(np.float16)
    x.reshape(-1)[:: 97] = 0
    return x


# one row; rows that are no multiple of a wave or a workgroup; head counts whose
# rows do not divide a workgroup; more pieces than threads (a second step per
# thread, and a last step that only some threads take)
@pytest.mark.parametrize("t,hq,hkv,d", [(1, 1, 1, 64), (3, 5, 5, 64), (7, 12, 12, 64), (33, 6, 3, 128), (2, 16, 2, 256),
                                        (3001, 8, 8, 128), (13001, 8, 8, 128)])
def test_rows(h, t, hq, hkv, d):
    rng = np.random.default_rng(t + d)
    q, k = _draw(rng, 1, t, hq, d), _draw(rng, 1, t, hkv, d)
    s = np.exp(rng.uniform(-2, 2, (hkv, d))).astype(np.float32)
    rows = np.unique(np.concatenate([np.arange(min(t, 24)), np.arange(max(0, t - 24), t), rng.integers(0, t, 40)]))
    for sv in (None, s):
        got = h.hifa4_quantize_qk(to_gpu(q), to_gpu(k), None if sv is None else to_gpu(sv))
        want = oatt.quantize_qk(q[0, rows], k[0, rows], sv)
        for g, w in zip(got, want):
            g = to_np(g)[rows]
            assert np.array_equal(g.view(w.dtype).reshape(w.shape), w)


# lengths around the 64-token groups and the half group a lane holds, an empty
# sequence, columns that do not fill a wave
@pytest.mark.parametrize("hkv,d,lens", [(1, 64, (1, 31, 32, 33)), (3, 64, (63, 64, 65, 0, 127)), (5, 128, (130,)),
                                        (2, 256, (96, 1))])
def test_tokens(h, hkv, d, lens):
    rng = np.random.default_rng(sum(lens) + d)
    v = _draw(rng, sum(lens), hkv, d)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    nb = (max(lens) + 63) // 64
    vc, vm = h.hifa4_quantize_v(to_gpu(v), cu_seqlens=to_gpu(cu), max_seqlen=max(lens))
    wc, wm = oatt.quantize_v(v, cu) if 0 not in lens else (None, None)
    vc, vm = to_np(vc), to_np(vm).view(np.uint32)
    at = 0
    for b, n in enumerate(lens):
        g = (n + 63) // 64
        if wc is None:
            one = oatt.quantize_v(v[cu[b]:cu[b + 1]], np.array([0, n])) if n else None
            c, m = one if n else (np.zeros((0,) + vc.shape[2:], np.uint8), np.zeros((0,) + vm.shape[2:], np.uint32))
        else:
            c, m = wc[at:at + g], wm[at:at + g]
            at += g
        assert np.array_equal(vc[b, :g], c) and np.array_equal(vm[b, :g], m)
        # groups past the end are the groups of 64 zeros: base 0, every E2 and E3 bit set
        assert not vc[b, g:].any() and np.all(vm[b, g:] == 0xFFFFFF00) and nb >= g


# fewer tokens than workgroups; runs that cross sequences; pieces that do not
# divide a workgroup; more pieces than threads
@pytest.mark.parametrize("n,s,hq,hkv,d", [(1, 1, 1, 1, 64), (3, 37, 10, 5, 64), (2, 700, 12, 12, 128), (5, 211, 8, 2, 256),
                                          (1, 9, 40, 40, 256)])
def test_calibration(h, n, s, hq, hkv, d):
    rng = np.random.default_rng(n * s + d)
    q, k = _draw(rng, n, s, hq, d), _draw(rng, n, s, hkv, d)
    k[..., 3] *= np.float16(9)
    for alpha in (-1.0, 0.5):
        sg, rep = h.hifa4_calibrate_smooth_qk(to_gpu(q), to_gpu(k), alpha)
        sw, want = osmooth.calibrate(q, k, hkv, alpha)
        assert rep["branch"] == want["branch"]
        assert abs(rep["rho_k"] - want["rho_k"]) <= 1e-9 * want["rho_k"]
        assert abs(rep["t_kq"] - want["t_kq"]) <= 1e-9 * want["t_kq"]
        ulps = np.abs(to_np(sg).view(np.int32).astype(np.int64) - sw.view(np.int32).astype(np.int64))
        assert ulps.max() <= 1


# the gate's reductions: no positive P99, one value, order statistics on both
# sides of a bin that another thread holds, more channels than threads
@pytest.mark.parametrize("kind,n,s,hkv,d", [("zero", 1, 3, 1, 64), ("one_value", 2, 50, 1, 64), ("split99", 1, 100, 1, 64),
                                            ("split99", 3, 77, 2, 128), ("normal", 40, 5, 10, 256)])
def test_calibration_gate(h, kind, n, s, hkv, d):
    rng = np.random.default_rng(n * s + hkv)
    q, k = _draw(rng, n, s, hkv, d), _draw(rng, n, s, hkv, d)
    if kind == "zero":
        k[:] = 0
    elif kind == "one_value":
        k[:] = np.float16(-2.5)
    elif kind == "split99":                       # the largest 1% from 2^-3 up: the two order statistics far apart
        k[:] = np.float16(0.0625)
        flat = k.reshape(-1)
        flat[:(flat.size - 1) // 100] = np.float16(7.0)
    for alpha in (-1.0, 0.25):
        sg, rep = h.hifa4_calibrate_smooth_qk(to_gpu(q), to_gpu(k), alpha)
        sw, want = osmooth.calibrate(q, k, hkv, alpha)
        assert rep["branch"] == want["branch"] and rep["alpha_used"] == want["alpha_used"]
        for name in ("rho_k", "t_kq"):            # float64 on both sides, a few roundings
            assert rep[name] == want[name] or abs(rep[name] - want[name]) <= 1e-12 * want[name], name
        ulps = np.abs(to_np(sg).view(np.int32).astype(np.int64) - sw.view(np.int32).astype(np.int64))
        assert ulps.max() <= 1
