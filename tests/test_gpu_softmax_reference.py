"""The reference of the decode kernels' softmax is the running maximum, so that the heaviest token's probability is a power of
two, which neither fp16 nor the product with an fp16 V scale rounds.  Logits that rise slowly over a workgroup's tiles, in jumps,
and fall, at V scales from 1 to 500; every weight that counts a new maximum; the mean error over the spread of the logits.
Against the fp64 oracle on the same bytes."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_mixed import _pack_both_mixed
from test_gpu_parity import B, _inputs, _np, _pack_both

pytestmark = pytest.mark.gpu

RISE = {"slow": lambda t: 30.0 * t, "steps": lambda t: 6.0 * np.floor(8 * t), "falls": lambda t: -20.0 * t, "flat": lambda t: 0.0 * t}


@pytest.mark.parametrize("v_scale", [1.0, 11.0, 13.0, 400.0])      # 2-bit V scales around 1.3, 15, 17, 530
@pytest.mark.parametrize("rise", sorted(RISE))
@pytest.mark.parametrize("hq,mixed", [(8, False), (16, False), (8, True)])
def test_reference_lags_and_catches_up(hq, mixed, rise, v_scale):
    print(f"[case] {hq} heads, channel-wise {mixed}, {rise}, V x {v_scale}", flush=True)
    b, rng, T = B(), np.random.default_rng(hq), 6000
    wl, inp, _ = _inputs("tiny", seq_lens=(T,), hq=hq)
    hkv = wl.hkv
    u = torch.randn(128, generator=torch.Generator().manual_seed(1))
    u /= u.norm()
    # logits (log2 domain) rise along the positions: q = 16 u + noise, k = noise + u x the rest
    lift = torch.from_numpy(RISE[rise](np.arange(T) / T) * (128 ** 0.5 / 1.4426950408889634 / 16.0)).float()
    K = inp["K"].float().view(hkv, T, 128) * 0.5 + lift[None, :, None] * u
    inp["K"] = K.to(torch.bfloat16).reshape(-1)
    inp["V"] = (inp["V"].float() * v_scale).to(torch.bfloat16)
    inp["q"] = (inp["q"].float() * 0.5 + 16.0 * u).to(torch.bfloat16)
    dev = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in inp.items()}
    bits = [rng.choice(np.array([2, 4, 8, 16], np.uint8), size=(hkv, T), p=[.6, .2, .1, .1])]
    if mixed:
        cache, ref = _pack_both_mixed(b, wl, inp, dev, bits, [rng.choice(np.array([4, 8], np.uint8), size=(hkv, 128))])
    else:
        cache, ref = _pack_both(b, wl, inp, dev, bits)
    out, lse = b.rdkv_decode_attn(cache, dev["q"])
    ref_out, ref_lse = O.decode(ref, _np(inp["q"]))
    got = out.cpu().numpy().astype(np.float64)
    err = np.abs(got - ref_out).max(axis=-1) / np.abs(ref_out).max(axis=-1)
    assert err.max() <= 2e-3, f"{err.max():.2e}"
    assert np.abs(lse.cpu().numpy() - ref_lse).max() <= 1e-4 * max(1.0, np.abs(ref_lse).max())
    cache.free()


@pytest.mark.parametrize("hq,mixed", [(8, False), (32, False), (64, False), (32, True), (64, True)])
@pytest.mark.parametrize("width", [2, 4, 8])
def test_a_new_maximum_is_not_rounded(hq, mixed, width):
    """One token of every tile counts, each more than all before it (the others' weights are below 2^-29): each is its wavefront's
    running maximum when it comes, so that p = 2^6 and its product with an fp16 V scale are exact in fp16.  What is left is fp32:
    a logit of up to 130 with a dozen roundings of 2^-24 moves its weight by 130 x 12 x 2^-24 x ln 2 = 6e-5 at most.  With a
    reference other than the running maximum p is rounded to 11 bits, and so is its product: up to 2^-11 + 2^-12 = 7e-4."""
    print(f"[case] {hq} heads, channel-wise {mixed}, {width} bits", flush=True)
    b, hkv, batch, tiles = B(), 8, 16, 100
    T, rng = 64 * tiles, np.random.default_rng(width)
    signs = torch.from_numpy(rng.choice([-1.0, 1.0], size=128)).float()
    K = torch.zeros(hkv, T, 128)
    at = torch.arange(tiles) * 64 + torch.from_numpy(rng.integers(0, 64, tiles))
    logits = 30.0 + torch.arange(tiles)                       # log2 domain, at q = signs
    K[:, at] = (logits * (128 ** 0.5 / 1.4426950408889634 / 128))[None, :, None] * signs
    V = torch.from_numpy(rng.standard_normal((hkv, T, 128))).float()
    K, V = K.to(torch.bfloat16).reshape(-1), V.to(torch.bfloat16).reshape(-1)
    q = signs.expand(batch, hq, 128).to(torch.bfloat16).contiguous()
    bits = [np.full((hkv, T), width, np.uint8)]
    bits_ch = [np.full((hkv, 128), width, np.uint8)]
    f = lambda x: x.float().numpy().reshape(hkv, T, 128)
    ref = O.build_cache_mixed([f(K)], [f(V)], bits, bits_ch) if mixed else O.build_cache_tokenwise([f(K)], [f(V)], bits)
    ref_out, _ = O.decode(ref, _np(q[:1]))
    cfg = b.Config([T] * batch, hq, hkv, k_mode=b.RDKV_K_CHANNELWISE if mixed else b.RDKV_K_TOKENWISE)
    cache = b.rdkv_pack(cfg, K.cuda().repeat(batch), V.cuda().repeat(batch), torch.from_numpy(bits[0]).reshape(-1).repeat(batch).cuda(),
                        torch.from_numpy(bits_ch[0]).reshape(-1).repeat(batch).cuda() if mixed else None)
    assert batch * hkv * tiles > 8 * cache.stats()["n_chunks"]      # a wavefront has more than one tile
    out, _ = b.rdkv_decode_attn(cache, q.cuda())
    err = np.abs(out.cpu().numpy().astype(np.float64) - ref_out).max(axis=-1) / np.abs(ref_out).max(axis=-1)
    print(f"[error] {err.max():.2e}", flush=True)
    assert err.max() <= 6e-5, f"{err.max():.2e}"
    cache.free()


# Both fp16 roundings (p, and p times a V scale) emulated on the CPU, 8 wavefronts of 16 tiles, running maximum per wavefront, the
# larger of 2 and 4 bits: 5.5e-4, 3.0e-4, 2.0e-4, 1.1e-4, 6.4e-5; times 1.5 for eight heads instead of many draws.  (With a
# reference that lags by up to 2^5: 5.2e-4, 4.7e-4, 4.1e-4, 3.1e-4, 2.2e-4.)
MEAN_ERROR = {1.0: 8.2e-4, 2.6: 4.5e-4, 4.0: 3.0e-4, 6.0: 1.6e-4, 9.0: 9.6e-5}


@pytest.mark.parametrize("hq", [32, 64])
@pytest.mark.parametrize("width", [2, 4])
@pytest.mark.parametrize("sigma", sorted(MEAN_ERROR))
def test_mean_error_over_the_spread_of_the_logits(sigma, width, hq):
    """Normal logits of spread sigma (log2 domain), normal values; rms error over rms output, mean over the heads."""
    b, hkv, batch, T = B(), 8, 16, 6400
    rng = np.random.default_rng(width)
    # a key of 128 equal channels: its groups have no range, so that it is held exactly at any width
    K = torch.from_numpy(np.repeat(rng.standard_normal((hkv, T, 1)), 128, axis=-1) * sigma / 1.4426950408889634 / 128 ** 0.5)
    V = torch.from_numpy(rng.standard_normal((hkv, T, 128)))
    K, V = K.to(torch.bfloat16).reshape(-1), V.to(torch.bfloat16).reshape(-1)
    q = torch.ones(batch, hq, 128).to(torch.bfloat16)
    bits = [np.full((hkv, T), width, np.uint8)]
    f = lambda x: x.float().numpy().reshape(hkv, T, 128)
    ref_out, _ = O.decode(O.build_cache_tokenwise([f(K)], [f(V)], bits), _np(q[:1]))
    cache = b.rdkv_pack(b.Config([T] * batch, hq, hkv), K.cuda().repeat(batch), V.cuda().repeat(batch),
                        torch.from_numpy(bits[0]).reshape(-1).repeat(batch).cuda())
    out, _ = b.rdkv_decode_attn(cache, q.cuda())
    d = out.cpu().numpy().astype(np.float64) - ref_out
    err = np.sqrt((d ** 2).mean(-1) / (ref_out ** 2).mean(-1)).mean()
    print(f"[case] sigma {sigma} {width} bits {hq} heads: {err:.2e}", flush=True)
    assert err <= MEAN_ERROR[sigma], f"{err:.2e}"
    cache.free()
