"""qadc_search_static (no allocation, static device scratch) against qadc_search, through the C ABI."""

import ctypes

import numpy as np
import pytest

from gpu_common import config1, to_gpu, gpu_us

pytestmark = pytest.mark.gpu


def _call_both(Q, L, torch, cb, queries, codes, R, init):
    nq, d = queries.shape
    m = cb.shape[0]
    n = codes.shape[0]
    dev = queries.device
    vp = ctypes.c_void_p
    stream = vp(torch.cuda.current_stream().cuda_stream)
    need = L.qadc_workspace_bytes(Q.QADC_WS_SEARCH, n, m, nq, R)
    ws = torch.zeros((max(need, 256),), dtype=torch.uint8, device=dev)
    out = [torch.full((nq, R), -7, dtype=torch.int32, device=dev) for _ in range(2)]
    dist = [torch.full((nq, R), 9, dtype=torch.uint8, device=dev) for _ in range(2)]
    ql = [torch.zeros((nq, m, 16), dtype=torch.uint8, device=dev) for _ in range(2)]
    rc = L.qadc_search(vp(cb.data_ptr()), d, m, vp(queries.data_ptr()), nq, vp(codes.data_ptr()), n, R, init,
                       255, 0, vp(out[0].data_ptr()), vp(dist[0].data_ptr()), vp(ql[0].data_ptr()),
                       vp(ws.data_ptr()), ws.numel(), stream)
    assert rc == 0, L.qadc_last_error()
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    rc = L.qadc_search_static(vp(cb.data_ptr()), d, m, vp(queries.data_ptr()), nq, vp(codes.data_ptr()), n, R,
                              init, 255, 0, vp(out[1].data_ptr()), vp(dist[1].data_ptr()), vp(ql[1].data_ptr()),
                              stream)
    assert rc == 0, L.qadc_last_error()
    torch.cuda.synchronize()
    assert torch.cuda.memory_allocated() == before
    assert torch.equal(ql[0], ql[1])
    assert torch.equal(out[0], out[1]) and torch.equal(dist[0], dist[1])
    return out[1], dist[1], ql[1]


def test_static_scratch_search_equals_workspace_search():
    import torch
    import paper_1704_07355_amd as Q
    from oracle import qadc_oracle as O
    L = Q.lib()
    assert L.qadc_static_scratch_bytes() == 32 << 20
    c = config1()
    cb, queries = to_gpu(c["codebooks"]), to_gpu(c["queries"])
    # a database long enough for the sampled bound and the barrier-free pass (tiled 4x)
    big = to_gpu(np.tile(c["codes"], (4, 1)))
    R, init = 100, 200
    # first call: one query over the long database; second call: smaller input (fewer codes, three
    # queries) on the same scratch, which the first call must have left clean
    i1, d1, q1 = _call_both(Q, L, torch, cb, queries[:1].contiguous(), big, R, init)
    small = big[:30_001].contiguous()
    i2, d2, q2 = _call_both(Q, L, torch, cb, queries[:3].contiguous(), small, R, init)
    # third call: a larger shape again (a batch over the long database): the array is laid out anew and
    # table data of the calls before must not be taken for control words
    i3, d3, q3 = _call_both(Q, L, torch, cb, queries[:16].contiguous(), big, R, init)
    # and against the oracle on the library's own tables (bit-exact)
    for (idx, dist, ql, codes_np, nq) in ((i1, d1, q1, np.tile(c["codes"], (4, 1)), 1),
                                          (i2, d2, q2, np.tile(c["codes"], (4, 1))[:30_001], 3),
                                          (i3, d3, q3, np.tile(c["codes"], (4, 1)), 16)):
        for iq in range(nq):
            wi, wd = O.top_r(O.scan_saturating(ql[iq].cpu().numpy(), codes_np), R, pad_dist=255)
            assert np.array_equal(idx[iq].cpu().numpy().view(np.uint32), wi)
            assert np.array_equal(dist[iq].cpu().numpy(), wd)


def test_static_scratch_rejects_sizes_beyond_the_array(monkeypatch):
    import paper_1704_07355_amd as Q
    L = Q.lib()
    # a launch shape whose per-query report regions exceed the array (8192 workgroups x 1024 keys x 8
    # bytes): refused before anything is enqueued or dereferenced
    monkeypatch.setenv("QADC_SCAN_WGS", "8192")
    n, m, R = 10_000_000, 16, 1024
    assert L.qadc_workspace_bytes(Q.QADC_WS_SEARCH, n, m, 1, R) > L.qadc_static_scratch_bytes()
    rc = L.qadc_search_static(None, 128, m, None, 1, None, n, R, 200, 255, 0, None, None, None, None)
    assert rc == Q.QADC_ENOMEM
    assert b"static" in L.qadc_last_error()


@pytest.mark.parametrize("n,m,nq,R", [(200_003, 16, 37, 1000), (700_001, 32, 35, 1000), (1_500_000, 64, 11, 1024)])
def test_static_scratch_calls_cut_into_unequal_sequences(n, m, nq, R):
    """A call of more queries than the array takes ends in a shorter launch sequence, which lays the scratch out its
    own way: it, and the call that follows, may not find anything of the one before."""
    import torch
    import paper_1704_07355_amd as Q
    L = Q.lib()
    rng = np.random.default_rng(n)
    cb = to_gpu(rng.uniform(0, 255, size=(m, 16, 2)).astype(np.float32))
    codes = to_gpu(rng.integers(0, 256, size=(n, m // 2), dtype=np.uint8))
    queries = to_gpu(rng.uniform(0, 255, size=(nq, 2 * m)).astype(np.float32))
    for _ in range(2):
        _call_both(Q, L, torch, cb, queries, codes, R, 200)


@pytest.mark.parametrize("m,n,nq", [(16, 10_000_000, 16), (32, 3_000_000, 64)])
def test_static_scratch_batches_are_not_cut_finer_than_they_were(m, n, nq):
    """The static array holds a batch of 16 queries over 10 M codes (and 16 of 64 at a time over 3 M, m = 32), whatever
    larger workspace a search would like better."""
    import torch
    import paper_1704_07355_amd as Q
    L = Q.lib()
    g = torch.Generator(device="cuda:0")
    g.manual_seed(m)
    cb = 30 * torch.randn((m, 16, 8), generator=g, device="cuda:0")
    codes = torch.randint(0, 256, (n, m // 2), generator=g, device="cuda:0", dtype=torch.uint8)
    queries = 30 * torch.randn((nq, 8 * m), generator=g, device="cuda:0")
    _call_both(Q, L, torch, cb, queries, codes, 100, 200)
    out = (torch.empty((nq, 100), dtype=torch.int32, device="cuda:0"), torch.empty((nq, 100), dtype=torch.uint8, device="cuda:0"))
    vp = ctypes.c_void_p

    def static():
        assert L.qadc_search_static(vp(cb.data_ptr()), 8 * m, m, vp(queries.data_ptr()), nq, vp(codes.data_ptr()), n, 100, 200, 255,
                                    0, vp(out[0].data_ptr()), vp(out[1].data_ptr()), None,
                                    vp(torch.cuda.current_stream().cuda_stream)) == 0

    ws = Q.qadc_workspace_init(torch.empty((Q.qadc_workspace_bytes(Q.QADC_WS_SEARCH, n, m, 16, 100),), dtype=torch.uint8,
                                           device="cuda:0"))
    q16 = queries[:16].contiguous()
    one = gpu_us(lambda: Q.qadc_search(cb, q16, codes, 100, 200, workspace=ws), reps=30)
    us = gpu_us(static, reps=30)
    assert us < 1.3 * one * (nq // 16), (us, one)
