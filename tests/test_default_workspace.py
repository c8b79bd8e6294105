"""Calls without a workspace of their own: which buffer each takes (on the CPU),
and that calls on two streams or two threads keep out of each other's (GPU)."""
import threading

import numpy as np
import pytest

import paper_2607_04302_amd as h
from paper_2607_04302_amd.workloads import small_case


def _fresh(monkeypatch, capturing=False):
    monkeypatch.setattr(h, "_scratch_buffers", threading.local())
    monkeypatch.setattr(h, "_capturing", lambda: capturing)


def test_a_buffer_per_stream_and_thread(monkeypatch):
    import torch
    _fresh(monkeypatch)
    dev = torch.device("cpu")
    a, b = h._scratch(1000, dev, 1), h._scratch(1000, dev, 2)
    assert a.data_ptr() != b.data_ptr()
    assert h._scratch(900, dev, 1) is a and h._scratch(1000, dev, 2) is b
    grown = h._scratch(5000, dev, 1)
    assert grown.numel() >= 5000 and h._scratch(1000, dev, 1) is grown and h._scratch(1000, dev, 2) is b
    other = []
    t = threading.Thread(target=lambda: other.append(h._scratch(1000, dev, 1)))
    t.start()
    t.join()
    assert other[0].data_ptr() != grown.data_ptr()


def test_the_buffers_are_bounded(monkeypatch):
    import torch
    _fresh(monkeypatch)
    for stream in range(100):
        h._scratch(256, torch.device("cpu"), stream)
    assert len(h._scratch_buffers.by_stream) == h._MAX_SCRATCH_STREAMS
    assert (None, 99) in h._scratch_buffers.by_stream


def test_a_captured_call_keeps_no_buffer(monkeypatch):
    import torch
    _fresh(monkeypatch)
    kept = h._scratch(256, torch.device("cpu"), 1)
    monkeypatch.setattr(h, "_capturing", lambda: True)
    assert h._scratch(256, torch.device("cpu"), 1) is not kept
    assert list(h._scratch_buffers.by_stream.values())[0] is kept


@pytest.mark.gpu
@pytest.mark.parametrize("threads", [False, True])
def test_two_streams_without_workspaces(threads):
    """Prefill and decode of different inputs and sizes side by side, none with
    a workspace: every output is that of the call alone."""
    import torch
    from _gpu_util import to_gpu
    jobs = []
    for i, lens in enumerate([(1000, 700, 64), (2000, 65)]):
        q, k, v, cu = small_case(heads_q=8, heads_kv=2, head_dim=128, seqlens=lens, seed=70 + i)
        q, k, v, cu_t = to_gpu(q), to_gpu(k), to_gpu(v), to_gpu(cu)
        kw = dict(cu_seqlens=cu_t, max_seqlen=max(lens))
        _, _, kc, km = h.hifa4_quantize_qk(None, k, None, **kw)
        vc, vm = h.hifa4_quantize_v(v, **kw)
        qd = q[torch.from_numpy(np.asarray(cu[1:], np.int64) - 1).cuda()].contiguous()
        jobs.append(lambda q=q, k=k, v=v, kc=kc, km=km, vc=vc, vm=vm, qd=qd, kw=kw:
                    (*h.hifa4_attention_fwd(q, k, v, **kw), *h.hifa4_decode_fwd(qd, kc, km, vc, vm, **kw)))
    want = [[x.clone() for x in job()] for job in jobs]
    torch.cuda.synchronize()
    got = [[], []]

    def work(i, stream):
        with torch.cuda.stream(stream):
            for _ in range(10):
                got[i].append(jobs[i]())

    streams = [torch.cuda.Stream() for _ in jobs]
    if threads:
        shared = torch.cuda.Stream()          # two threads whose launches interleave on one stream
        runs = [threading.Thread(target=work, args=(i, shared)) for i in range(2)]
        for t in runs:
            t.start()
        for t in runs:
            t.join()
    else:
        for _ in range(5):
            for i in range(2):
                with torch.cuda.stream(streams[i]):
                    got[i].append(jobs[i]())
    torch.cuda.synchronize()
    for i in range(2):
        assert got[i]
        for out in got[i]:
            assert all(torch.equal(a, b) for a, b in zip(out, want[i])), i


@pytest.mark.gpu
def test_captured_without_workspace_then_larger_calls():
    """A call captured without a workspace replays correctly after larger eager
    calls on the same stream have had theirs replaced."""
    import torch
    from _gpu_util import to_gpu
    q, k, v, _ = (to_gpu(x) if x is not None else None for x in
                  small_case(heads_q=4, heads_kv=2, head_dim=128, seqlens=(300,), seed=75))
    kw = dict(cu_seqlens=to_gpu(np.array([0, 300], np.int32)), max_seqlen=300)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        want = [x.clone() for x in h.hifa4_attention_fwd(q, k, v, **kw)]
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        got = h.hifa4_attention_fwd(q, k, v, **kw)
    big = torch.randn(1, 3000, 4, 128, device="cuda", dtype=torch.float16)
    for _ in range(3):
        with torch.cuda.stream(side):
            h.hifa4_attention_fwd(big, big, big)
        junk = torch.full((32 << 20,), 7, dtype=torch.uint8, device="cuda")
        for x in got:
            x.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, want))
        del junk
