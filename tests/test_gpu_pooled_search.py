"""rdkv_compress pools the weights inside the search's first launch, the staged calls in a launch of its own: the same bit maps,
multipliers and step counts, at the edges of the units a thread, a workgroup and a slice hold, for several windows, and with
weights down to where fp32 ends (logits hundreds of powers of two apart)."""
import numpy as np
import pytest
import torch

from test_gpu_parity import B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens", [(33, 64), (1000, 37), (4093, 4096), (4097,), (16384, 16381), (32768, 9), (32769, 40), (50001,), (70000, 131072)])
@pytest.mark.parametrize("pool", [1, 3, 5, 15])
@pytest.mark.parametrize("spread", [1.0, 30.0])
def test_fused_pooling(lens, pool, spread):
    print(f"[case] {lens} window {pool} spread {spread}", flush=True)
    b, hkv = B(), 2
    gen = torch.Generator(device="cuda").manual_seed(sum(lens))
    K, V = (torch.randn(sum(lens) * hkv * 128, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    Q = spread * torch.randn((len(lens), hkv, 4, 128), generator=gen, device="cuda", dtype=torch.bfloat16)
    cfg = b.Config(lens, hkv, hkv, budget_bits=[1.5] * len(lens), s_obs=4, pool_kernel=pool)
    cache = b.rdkv_compress(cfg, K, V, Q)
    w, _ = b.rdkv_weights(cfg, K, Q)
    bits, _, lam, iters = b.rdkv_allocate_info(cfg, w)
    assert np.array_equal(cache.export(b.RDKV_EXPORT_BITS_TOK, np.uint8), bits.cpu().numpy())
    assert np.array_equal(cache.export(b.RDKV_EXPORT_LAMBDA, np.float64), lam.cpu().numpy().reshape(-1), equal_nan=True)
    assert np.array_equal(cache.export(b.RDKV_EXPORT_ITERATIONS, np.int32), iters.cpu().numpy().reshape(-1))
    cache.free()


# Windows without a weight above zero, whole ones and next to the smallest and to ordinary sums in the same four: the pooling's short way
# takes the zeros, and its division the rest.
@pytest.mark.parametrize("lens", [(64, 1000), (4096, 4097), (8190,), (20000, 33), (32768,), (50001,)])
@pytest.mark.parametrize("pool", [3, 5, 15])
def test_windows_of_zeros(lens, pool):
    print(f"[case] {lens} window {pool}", flush=True)
    b, hkv = B(), 2
    gen = torch.Generator(device="cuda").manual_seed(sum(lens) + pool)
    K, V = (torch.randn(sum(lens) * hkv * 128, generator=gen, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    Q = 300.0 * torch.randn((len(lens), hkv, 4, 128), generator=gen, device="cuda", dtype=torch.bfloat16)
    cfg = b.Config(lens, hkv, hkv, budget_bits=[0.2] * len(lens), s_obs=4, pool_kernel=pool)
    w, _ = b.rdkv_weights(cfg, K, Q)
    raw, _ = b.rdkv_weights(b.Config(lens, hkv, hkv, budget_bits=[0.2] * len(lens), s_obs=4, pool_kernel=1), K, Q)
    off = 0
    for T in lens:                       # the pooled weights: fp32 sums in the window's order, IEEE quotients
        x = np.pad(raw[off:off + hkv * T].cpu().numpy().reshape(hkv, T), ((0, 0), (pool // 2, pool // 2)))
        s = np.zeros((hkv, T), np.float32)
        for k in range(pool):
            s = s + x[:, k:k + T]
        assert (s == 0).any() and (s > 0).any()
        assert np.array_equal(w[off:off + hkv * T].cpu().numpy().reshape(hkv, T), s / np.float32(pool))
        off += hkv * T
    cache = b.rdkv_compress(cfg, K, V, Q)
    bits, _, lam, iters = b.rdkv_allocate_info(cfg, w)
    assert np.array_equal(cache.export(b.RDKV_EXPORT_BITS_TOK, np.uint8), bits.cpu().numpy())
    assert np.array_equal(cache.export(b.RDKV_EXPORT_LAMBDA, np.float64), lam.cpu().numpy().reshape(-1), equal_nan=True)
    assert np.array_equal(cache.export(b.RDKV_EXPORT_ITERATIONS, np.int32), iters.cpu().numpy().reshape(-1))
    cache.free()
