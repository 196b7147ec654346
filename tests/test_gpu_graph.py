"""The whole path (encode, decode, fused attention) enqueues plain kernel launches only, so a caller can
record it into a HIP graph.  The graph is replayed several times with eager work in between, and every
replay must reproduce the eager bytes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2605_27646_amd as hq
import workloads

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def test_graph_replays_match_eager():
    B, H, T, S, G = 1, 4, 700, 64, 4
    wl = workloads.Workload("graph", 900, 1, B, H, T, 128, S, sigma_g=0.8)
    k = workloads.make_tensor(wl, 0, 0, "cpu").to(DEV)
    v = workloads.make_tensor(wl, 0, 1, "cpu").to(DEV)
    cb = hq.hqmq_build_codebooks(1, 1, H, S).to(DEV)
    sec_k, sec_v = cb[0, 0].contiguous(), cb[0, 1].contiguous()
    params = hq.params_for(k, S)
    ek, ev = hq.alloc_encoded(params, DEV), hq.alloc_encoded(params, DEV)
    ws = hq.alloc_batch_workspace(params, 2, DEV)
    batch = hq.EncodeBatch(params, [k, v], [sec_k, sec_v], [ek, ev], ws)
    ok, ov = torch.empty_like(k), torch.empty_like(v)
    dec = hq.DecodeBatch(params, [ek, ev], [sec_k, sec_v], [ok, ov])
    q = torch.randn(B, H * G, 128, generator=torch.Generator().manual_seed(3)).to(torch.float16).to(DEV)
    o = torch.empty_like(q)
    aws = torch.empty(hq.hqmq_attend_workspace_bytes(params, H * G), dtype=torch.uint8, device=DEV)
    o2 = torch.empty_like(q)
    lse = torch.empty(B, H * G, dtype=torch.float32, device=DEV)
    vis = torch.randint(0, T + 1, (B, H * G), generator=torch.Generator().manual_seed(4), dtype=torch.int32).to(DEV)
    aws2 = torch.empty_like(aws)

    es = hq.alloc_encoded(params, DEV)          # K once more through the entry point that takes no workspace

    def path():
        hq.hqmq_encode_static(params, k, sec_k, es)
        hq.hqmq_encode_batch(batch)
        hq.hqmq_decode_batch(dec)
        hq.hqmq_attend(params, q, 0.09, ek, sec_k, ev, sec_v, o, aws)
        hq.hqmq_attend_masked(params, q, 0.09, ek, sec_k, ev, sec_v, vis, o2, aws2, lse)

    def snapshot():
        torch.cuda.synchronize()
        return [t.clone() for t in (es.codes, es.row_off, es.n_outliers, es.status,
                                    ek.codes, ek.flags, ek.row_off, ek.n_outliers, ev.codes, ok.view(torch.int16),
                                    ov.view(torch.int16), o.view(torch.int16), o2.view(torch.int16),
                                    lse.view(torch.int32))]

    def scrub():
        for t in (ek.codes, ek.flags, ek.row_off, ev.codes, ek.n_outliers, es.codes, es.row_off, es.n_outliers, es.status):
            t.fill_(-1)
        for t in (ok, ov, o, o2, lse):
            t.fill_(float("nan"))
        ws.fill_(0x77)
        aws.fill_(0x77)
        aws2.fill_(0x77)

    hq.hqmq_init()                              # per-device set-up outside any capture
    path()
    want = snapshot()
    assert int(ek.n_outliers[-1]) > 0
    assert torch.equal(es.codes, ek.codes) and torch.equal(es.row_off, ek.row_off)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        path()                                  # warm-up on the capture stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        path()
    for rep in range(3):
        scrub()
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for a, b in zip(got, want):
            assert torch.equal(a, b), rep
        # eager work of the program's own between the replays
        path()
        torch.cuda.synchronize()


@pytest.mark.parametrize("n,B,H,T,D,S,given", [
    (2, 1, 2, 6000, 128, 64, False),   # sweep with the box index beside it
    (1, 2, 3, 1537, 100, 96, False),   # the same for any row length, decode included
    (1, 2, 2, 1100, 128, 16, False),   # sweep alone, matrix screen
    (3, 1, 8, 1, 128, 256, True),      # rows of a generation step: one launch
    (3, 2, 8, 5, 96, 48, True),        # two launches
    (2, 1, 2, 5000, 128, 128, True),   # thresholds known: the index in a launch of its own
])
def test_graph_replays_of_the_encodes_forms(n, B, H, T, D, S, given):
    xs = [workloads.make_tensor(workloads.Workload("graph", 910 + i, 1, B, H, T, D, S, sigma_g=0.8), 0, 0, "cpu").to(DEV)
          for i in range(n)]
    cb = hq.hqmq_build_codebooks(1, n, H, S).to(DEV)
    secs = [cb[i, 0].contiguous() for i in range(n)]
    params = hq.params_for(xs[0], S)
    encs = [hq.alloc_encoded(params, DEV, outlier_capacity=B * H * T * ((D + 3) // 4)) for _ in range(n)]
    ws = hq.alloc_batch_workspace(params, n, DEV)
    batch = hq.EncodeBatch(params, xs, secs, encs, ws)
    thrs = hq.ThresholdBatch(batch, [torch.full((H,), 6.0, dtype=torch.float64, device=DEV)] * n) if given else None
    outs = [torch.empty_like(x) for x in xs]
    dec = hq.DecodeBatch(params, encs, secs, outs)

    def path():
        if given:
            hq.hqmq_encode_batch_given_thresholds(batch, thrs)
        else:
            hq.hqmq_encode_batch(batch)
        hq.hqmq_decode_batch(dec)

    def state():
        return [t for e, o in zip(encs, outs) for t in (e.codes, e.sigma, e.flags, e.row_off, e.n_outliers, e.status, o)]

    def snapshot():
        torch.cuda.synchronize()
        return [(t.view(torch.int16) if t.dtype == torch.float16 else t).clone() for t in state()]

    hq.hqmq_init()
    path()
    want = snapshot()
    assert all(int(e.n_outliers[-1]) > 0 for e in encs)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        path()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        path()
    for rep in range(3):
        for t in state():
            t.fill_(-1)
        ws.fill_(0x77)
        torch.cuda.synchronize()
        graph.replay()
        for a, b in zip(snapshot(), want):
            assert torch.equal(a, b), rep
        path()
        torch.cuda.synchronize()


@pytest.mark.parametrize("raw", [True, False])
def test_calls_go_to_the_current_stream(raw, monkeypatch):
    """The stream that a call without one takes is torch's current one, from the handle that this torch gives directly or, where
    it does not, from a Stream object: on the default stream, on another, in another thread and while a graph is captured."""
    import threading

    from paper_2605_27646_amd import binding
    if not raw:
        monkeypatch.setattr(binding, "_raw_stream", None)
    elif binding._raw_stream is None:
        pytest.skip("this torch has no handle without a Stream object")

    def agrees():
        return binding._stream_ptr(None) == torch.cuda.current_stream().cuda_stream

    assert agrees()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert agrees() and binding._stream_ptr(None) == side.cuda_stream
        seen = []
        t = threading.Thread(target=lambda: seen.append((agrees(), binding._stream_ptr(None))))
        t.start()
        t.join()
        assert seen[0][0] and seen[0][1] != side.cuda_stream
        assert binding._stream_ptr(side) == side.cuda_stream
    assert agrees() and binding._stream_ptr(None) != side.cuda_stream
    graph = torch.cuda.CUDAGraph()
    buf = torch.zeros(4, device="cuda:0")
    with torch.cuda.graph(graph):
        assert agrees()
        buf.add_(1.0)
    graph.replay()
    torch.cuda.synchronize()
