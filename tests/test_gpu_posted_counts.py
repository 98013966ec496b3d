"""rdkv_compress on items of up to 32K tokens learns the tier counts (and the channels' widths) from words that the search posts to
the host; rdkv_pack counts the bit map.  Both give the same cache: searches, maps that no search makes (everything kept, nothing
kept), the shortest sequences, both sides of 32K tokens, more items than the staging ring has room for."""
import numpy as np
import pytest
import torch

from test_gpu_parity import B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["token", "channel", "per_channel"])
@pytest.mark.parametrize("lens,budgets", [
    ((4, 33, 64), (1.0, 16.0, 0.01)), ((700, 5, 1025), (2.0, 1.0, 0.5)), ((4096, 4097), (16.0, 0.001)), ((8192, 8193, 9), (0.7, 3.0, 2.0)),
    ((32768, 16384), (1.0, 1.0)), ((32769, 5), (1.0, 1.0)), (tuple(4 + i % 7 for i in range(4200)), tuple(0.5 + i % 5 for i in range(4200)))])
def test_compress_is_the_staged_calls(lens, budgets, mode):
    b, hkv = B(), 8 if len(lens) > 1000 else 2
    print(f"[case] {len(lens)} sequences, {lens[:3]}, {mode}", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(sum(lens))
    K, V = (torch.randn(sum(lens) * hkv * 128, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    Q = torch.randn((len(lens), hkv, 4, 128), generator=gen, device="cuda", dtype=torch.bfloat16)
    kw = {} if mode == "token" else {"k_mode": b.RDKV_K_CHANNELWISE, "k_scale_per_channel": int(mode == "per_channel")}
    cfg = b.Config(lens, hkv, hkv, budget_bits=list(budgets), s_obs=4, **kw)
    whole = b.rdkv_compress(cfg, K, V, Q)
    w, w_ch = b.rdkv_weights(cfg, K, Q, want_channel=mode != "token")
    staged = b.rdkv_pack(cfg, K, V, *b.rdkv_allocate(cfg, w, w_ch))
    torch.cuda.synchronize()
    a, c = whole.stats(), staged.stats()
    assert all(a[k] == c[k] for k in ("rows", "evicted", "stored_bytes", "arena_bytes", "n_chunks"))
    for what in (b.RDKV_EXPORT_ARENA, b.RDKV_EXPORT_BITS_TOK):
        assert np.array_equal(whole.export(what, np.uint8), staged.export(what, np.uint8))
    whole.free()
    staged.free()
