"""The staged calls recorded in a HIP graph: their host tables go with the graph, so that a replay neither depends on the
staging memory the call used at capture nor touches it, and the calls that wait for the stream record nothing."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from test_gpu_parity import B

pytestmark = pytest.mark.gpu


def _batch(batch, hkv, T, s_obs, seed):
    rng = torch.Generator().manual_seed(seed)
    K = torch.randn(batch * hkv * T * 128, generator=rng).to(torch.bfloat16).cuda()
    Q = torch.randn((batch, hkv, s_obs, 128), generator=rng).to(torch.bfloat16).cuda()
    return K, Q


@pytest.mark.parametrize("mixed", [False, True])
# 32 bytes a sequence: along with each launch up to 32 sequences; then a table, which a graph takes 3 KB a launch: one launch, three,
# 42; and beyond half the staging ring (1 MB), where an eager call has memory of its own that it waits for and gives back
@pytest.mark.parametrize("batch,hkv,T,s_obs", [(2, 8, 700, 32), (32, 2, 64, 32), (33, 2, 64, 32), (90, 8, 64, 32), (200, 2, 64, 32),
                                               (4000, 8, 33, 32), (33000, 1, 9, 4)])
def test_replays_of_the_staged_calls(batch, hkv, T, s_obs, mixed):
    b = B()
    print(f"[case] captured weights and allocation, {batch} x {T}, {hkv} heads, channel-wise {mixed}", flush=True)
    K, Q = _batch(batch, hkv, T, s_obs, batch)
    budgets = [0.5 + s % 4 for s in range(batch)]
    cfg = b.Config([T] * batch, hkv, hkv, budget_bits=budgets, s_obs=s_obs, **b.torch_allocator_hooks(),
                   **({"k_mode": b.RDKV_K_CHANNELWISE} if mixed else {}))
    # unrelated work whose tables go once round the ring between two replays
    other_batch = 1100
    oK, oQ = _batch(other_batch, 8, 40, 32, 7)
    other = b.Config([40] * other_batch, 8, 8, budget_bits=[2.0] * other_batch, s_obs=32, **b.torch_allocator_hooks())
    oq = oQ[:, :, 0].contiguous()

    def unrelated():
        outs = []
        for _ in range(3):
            cache = b.rdkv_compress(other, oK, oK, oQ)
            outs.append(b.rdkv_decode_attn(cache, oq)[0].clone())
            torch.cuda.synchronize()
            cache.free()
        return outs

    def staged():
        w_tok, w_ch = b.rdkv_weights(cfg, K, Q, want_channel=mixed)
        bits_tok, bits_ch = b.rdkv_allocate(cfg, w_tok, w_ch)
        return [x for x in (w_tok, w_ch, bits_tok, bits_ch) if x is not None]

    eager, expected = staged(), unrelated()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        recorded = staged()
    for _ in range(4):
        for x in recorded:
            x.zero_()
        torch.cuda.synchronize()
        graph.replay()
        got = unrelated()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(recorded, eager))
        assert all(torch.equal(x, y) for x, y in zip(got, expected))


def test_calls_that_wait_are_refused_under_capture():
    b, hkv, T = B(), 2, 300
    K, Q = _batch(1, hkv, T, 32, 1)
    cfg = b.Config([T], hkv, hkv, budget_bits=[2.0], s_obs=32, **b.torch_allocator_hooks())
    bits = torch.from_numpy(np.random.default_rng(1).choice(np.array([0, 2, 4], np.uint8), size=hkv * T)).cuda()
    q = Q[:, :, 0].contiguous()
    cache, tailed = b.rdkv_pack(cfg, K, K, bits), b.rdkv_pack(cfg, K, K, bits)
    b.rdkv_cache_reserve_tail(tailed, 64)
    row = K[:hkv * 128].view(1, hkv, 128)
    for _ in range(40):
        b.rdkv_cache_append(tailed, row, row)
    before, _ = b.rdkv_decode_attn(tailed, q)
    out, lse = torch.empty_like(before), torch.empty_like(before[..., 0])
    tail_cfg = b.Config([40], hkv, hkv, budget_bits=[2.0], s_obs=32, **b.torch_allocator_hooks())
    calls = [lambda: b.rdkv_pack(cfg, K, K, bits), lambda: b.rdkv_compress(cfg, K, K, Q), lambda: b.rdkv_calibrate_eps(cfg, K, K),
             lambda: b.rdkv_cache_reserve_tail(cache, 8), lambda: b.rdkv_cache_tail_len_sync(tailed),
             lambda: b.rdkv_cache_rebudget_tail(tailed, tail_cfg, Q)]
    status = []
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for call in calls:
            try:
                call()
                status.append(0)
            except b.RdkvError as e:
                status.append(e.status)
        b.rdkv_decode_attn(tailed, q, out, lse)          # the capture goes on
    assert status == [5] * len(calls)
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, before)
    for call in calls:                                   # and outside of one they all still run
        call()
    torch.cuda.synchronize()


def test_another_thread_calls_while_this_one_captures():
    """A staged call without allocator hooks, whose scratch is larger than what the library holds so far, on a stream and a
    thread of its own beside a capture: neither disturbs the other."""
    b, hkv = B(), 2
    K, Q = _batch(1, hkv, 300, 32, 1)
    cfg = b.Config([300], hkv, hkv, budget_bits=[2.0], s_obs=32)
    cache = b.rdkv_compress(cfg, K, K, Q)
    q = Q[:, :, 0].contiguous()
    expected, _ = b.rdkv_decode_attn(cache, q)
    T = 40000
    big_K, big_Q = _batch(4, 8, T, 32, 2)
    big = b.Config([T] * 4, 8, 8, budget_bits=[1.0] * 4, s_obs=32)
    w = torch.empty(4 * 8 * T, dtype=torch.float32, device="cuda")
    out, lse = torch.empty_like(expected), torch.empty_like(expected[..., 0])
    side, status = torch.cuda.Stream(), []

    def call():
        status.append(b.lib.rdkv_weights(big.ref(), big_K.data_ptr(), big_Q.data_ptr(), w.data_ptr(), None,
                                         ctypes.c_void_p(side.cuda_stream)))

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        b.rdkv_decode_attn(cache, q, out, lse)
        thread = threading.Thread(target=call)
        thread.start()
        thread.join()
    torch.cuda.synchronize()
    assert status == [0]
    assert torch.equal(w, b.rdkv_weights(big, big_K, big_Q)[0])
    for _ in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, expected)
    cache.free()
