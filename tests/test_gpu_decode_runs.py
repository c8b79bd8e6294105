"""Decode step: every way a call's blocks become runs.  Run lengths of 1 to 8
blocks, numbered over the sequences' own lengths (up to 256 sequences, the
prefix sum over the batch in one to four steps) or over the longest one (more
sequences, or no cu_seqlens), last blocks of 1 to 64 keys, empty sequences, one
to eight waves per workgroup; each case asserts the plan that it stands for.
Every P^ code of the sampled rows bit-exact against the oracle, O and LSE
within the parity bar and the same bits without the P^ dump.  Then lengths that
grow under a captured call, waits that give up, and calls on two streams."""
import numpy as np
import pytest

from paper_2607_04302_amd.workloads import small_case

from _gpu_util import check_close, to_gpu, to_np
from test_decode_plan import load_plan, plan
from test_gpu_decode import _build_cache, _decode_and_compare, _say, h  # noqa: F401  (h: the library fixture)

pytestmark = pytest.mark.gpu


def _lens(n, lo, hi, seed, empty=()):
    x = np.random.default_rng(seed).integers(lo, hi + 1, n)
    x[list(empty)] = 0
    return tuple(int(v) for v in x)


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    lib = load_plan(tmp_path_factory.mktemp("plan"))

    def of(lens, max_seqlen, d, hq, hkv, cu=True):
        p = plan(lib, len(lens), hq, hkv, d, -(-max_seqlen // 64), sum(lens) if cu else -1)
        return p["bps"], p["packed"], p["waves"]
    return of


# want: blocks per run, runs numbered over the own lengths, waves per workgroup
@pytest.mark.parametrize("lens,d,hq,hkv,seqs,kv_heads,want", [
    ((64, 65, 127, 128, 1, 63), 128, 8, 2, None, None, (2, 1, 1)),                  # every kind of last block
    (_lens(70, 1, 200, 1, empty=(0, 63, 64)), 64, 2, 1, [1, 62, 65, 69], None, (1, 1, 1)),     # two prefix-sum steps
    (_lens(200, 1, 90, 2, empty=(199,)), 128, 4, 1, [0, 127, 128, 198], None, (2, 1, 1)),      # four steps
    (_lens(300, 1, 150, 3, empty=(5, 299)), 64, 1, 1, [0, 4, 256, 298], None, (3, 0, 1)),      # above 256 sequences
    ((2999, 3300, 70, 3265), 64, 64, 64, [0, 2, 3], [0, 63], (4, 1, 8)),
    ((4001, 4100, 3900, 4096, 64), 64, 64, 64, [1, 4], [5], (7, 1, 8)),
    ((5000, 4097, 63), 256, 16, 16, [0, 1, 2], [0, 15], (2, 1, 4)),                 # D = 256
    ((3000, 2047), 256, 40, 8, [0, 1], [7], (2, 1, 1)),                             # two rows per lane, GQA x5
])
def test_decode_run_shapes(h, planner, lens, d, hq, hkv, seqs, kv_heads, want):  # noqa: F811
    assert planner(lens, max(lens), d, hq, hkv) == want
    _, k, v, cu = small_case(heads_q=hkv, heads_kv=hkv, head_dim=d, seqlens=lens, seed=41)
    qd = np.random.default_rng(42).standard_normal((len(lens), hq, d)).astype(np.float16)
    s = np.exp(np.random.default_rng(43).uniform(-1, 1, (hkv, d))).astype(np.float32)
    _say("decode runs", len(lens), max(lens), d, hq, hkv)
    _decode_and_compare(h, qd, k, v, cu, s, max(lens), seqs=seqs, kv_heads=kv_heads)


@pytest.mark.parametrize("blocks,d,hq", [(1, 128, 4), (2, 64, 8), (3, 256, 1), (4, 128, 8), (5, 64, 2), (6, 256, 2),
                                         (7, 128, 1), (8, 64, 4)])
def test_decode_run_lengths(h, planner, blocks, d, hq):  # noqa: F811
    """Every run length, by the longest sequence (128 runs of it): in calls of
    two packed sequences, and of one sequence without cu_seqlens (its runs of
    one block are those of one block in all)."""
    lens = (8192 * blocks - 3, 130)
    assert planner(lens, lens[0], d, hq, 1)[:2] == (blocks, 1)
    _, k, v, cu = small_case(heads_q=1, heads_kv=1, head_dim=d, seqlens=lens, seed=46)
    qd = np.random.default_rng(47).standard_normal((2, hq, d)).astype(np.float16)
    _say("decode run lengths", blocks, d, hq)
    _decode_and_compare(h, qd, k, v, cu, None, lens[0])
    n = lens[0] if blocks > 1 else 60
    assert planner((n,), n, d, hq, 1, cu=False)[:2] == (blocks, 0)
    _decode_and_compare(h, qd[:1], k[None, :n], v[None, :n], None, None, n)


@pytest.mark.parametrize("norm", ["preorder", "inconsistent"])
def test_decode_max_seqlen_above_every_length(h, norm):  # noqa: F811
    """max_seqlen as an upper bound (a preallocated cache): the grid follows
    the cached tokens, the V^ cache and the P^ dump the bound."""
    lens = (700, 0, 65, 1)
    _, k, v, cu = small_case(heads_q=2, heads_kv=2, head_dim=128, seqlens=lens, seed=44)
    qd = np.random.default_rng(45).standard_normal((len(lens), 8, 128)).astype(np.float16)
    _say("decode bound above lengths", norm)
    _decode_and_compare(h, qd, k, v, cu, None, 5000, norm=norm)


@pytest.mark.parametrize("captured,grown,d,hq,hkv", [
    ((64, 1, 30), (1500, 64, 2000), 128, 8, 2),              # planned runs of 1 become 6, several per workgroup
    ((1, 1), (9000, 8191), 64, 8, 8),                        # 2 become 8, 34 runs in 2 workgroups
    ((200,) * 70, (700,) * 35 + (65,) * 35, 64, 2, 1),       # 1 become 4, two steps of the prefix sum
    ((5, 0, 3), (300, 1200, 0), 256, 8, 1),                  # 1 become 3; a sequence appears, another empties
])
def test_decode_captured_lengths_grow(h, captured, grown, d, hq, hkv):  # noqa: F811
    """A captured step replayed over lengths that have grown in place past the
    captured number of tokens, within max_seqlen: every run is computed, P^
    equals the eager call on the new lengths bit for bit, O and LSE agree to
    fp32 rounding (the runs may be cut elsewhere)."""
    import torch
    cap = max(grown)
    _, k, v, cu = small_case(heads_q=hkv, heads_kv=hkv, head_dim=d, seqlens=grown, seed=51)
    qd = to_gpu(np.random.default_rng(52).standard_normal((len(grown), hq, d)).astype(np.float16))
    kc, km, vc, vm, cu_new = _build_cache(h, k, v, None, cu, cap)
    want = h.hifa4_decode_fwd(qd, kc, km, vc, vm, cu_seqlens=cu_new, max_seqlen=cap, debug_p=True)
    cu_t = to_gpu(np.concatenate([[0], np.cumsum(captured)]).astype(np.int32))
    t = int(sum(captured))
    kw = dict(cu_seqlens=cu_t, max_seqlen=cap, workspace=h.Workspace(), debug_p=True)
    _say("decode captured lengths grow", len(grown), t, sum(grown), d)
    h.hifa4_decode_fwd(qd, kc[:t], km[:t], vc, vm, **kw)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        got = h.hifa4_decode_fwd(qd, kc[:t], km[:t], vc, vm, **kw)
    for step in range(3):
        cu_t.copy_(cu_new)
        for x in got:
            x.zero_()
        graph.replay()
        torch.cuda.synchronize()
        live = [b for b, n in enumerate(grown) if n]
        assert torch.equal(got[2], want[2]) and torch.equal(got[3], want[3]), step
        # two roundings of fp16 outputs apart; LSE: a few fp32 roundings of values below 2^5
        check_close(to_np(got[0][live]), to_np(want[0][live]), atol=1e-4, rtol=2e-3, what="O")
        check_close(to_np(got[1][:, live]), to_np(want[1][:, live]), atol=2e-5, rtol=0, what="LSE")
        h.hifa4_decode_fwd(qd, kc, km, vc, vm, cu_seqlens=cu_new, max_seqlen=cap)      # eager work between
        torch.cuda.synchronize()


def _case(h, lens, d, hq, hkv, seed):  # noqa: F811
    _, k, v, cu = small_case(heads_q=hkv, heads_kv=hkv, head_dim=d, seqlens=lens, seed=seed)
    qd = to_gpu(np.random.default_rng(seed).standard_normal((len(lens), hq, d)).astype(np.float16))
    return qd, _build_cache(h, k, v, None, cu, max(lens))


@pytest.mark.parametrize("lens,d,hq,hkv", [
    ((700, 65, 64, 1), 128, 8, 2),                   # runs of one block
    ((4096, 300, 4001), 64, 16, 2),                  # GQA x8
    ((16384,) * 8, 128, 32, 8),                      # longer runs, the later ones behind 50 others
    ((16384, 130), 64, 64, 64),
    ((5000, 2047), 256, 16, 16),
    ((3000, 129), 256, 40, 8),                       # D = 256, GQA x5
])
def test_decode_without_published_maxima(h, lens, d, hq, hkv):  # noqa: F811
    """No run maximum is published and every wait gives up after 16 polls: each
    run scores the blocks before it itself, and every output is the same bits."""
    import torch
    qd, (kc, km, vc, vm, cu_t) = _case(h, lens, d, hq, hkv, 61)
    for norm in (h.NORM_PREORDER, h.NORM_INCONSISTENT):
        kw = dict(cu_seqlens=cu_t, max_seqlen=max(lens), norm=norm)
        _say("decode without published maxima", lens, d, hq, hkv, norm)
        for dump in (False, True):
            want = h.hifa4_decode_fwd(qd, kc, km, vc, vm, debug_p=dump, **kw)
            got = h.hifa4_decode_fwd(qd, kc, km, vc, vm, debug_p=dump, test_no_publish=2, **kw)
            torch.cuda.synchronize()
            assert not torch.isnan(want[0]).any()
            assert all(torch.equal(a, b) for a, b in zip(got, want)), dump


def test_decode_on_two_streams(h):  # noqa: F811
    """Two calls that each fill the GPU, side by side on two streams with a
    workspace each: whatever workgroups the one keeps off the GPU while its own
    wait, both give the bits of a call alone."""
    import torch
    cases = [_case(h, (16384,) * 8, 128, 32, 8, 62), _case(h, (9000, 16000, 16384, 300) * 4, 128, 32, 8, 63)]
    kw = [dict(cu_seqlens=c[1][4], max_seqlen=16384, workspace=h.Workspace()) for c in cases]
    want = [[x.clone() for x in h.hifa4_decode_fwd(c[0], *c[1][:4], **k)] for c, k in zip(cases, kw)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]
    got = [[], []]
    _say("decode on two streams")
    for _ in range(20):
        for i, st in enumerate(streams):
            with torch.cuda.stream(st):
                got[i].append(h.hifa4_decode_fwd(cases[i][0], *cases[i][1][:4], **kw[i]))
    torch.cuda.synchronize()
    for i in range(2):
        for o, l in got[i]:
            assert torch.equal(o, want[i][0]) and torch.equal(l, want[i][1]), i
