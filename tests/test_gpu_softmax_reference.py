"""The decode kernels' softmax takes a logit of a while ago for its reference as long as none exceeds it by 2^5: logits that rise
slowly over a workgroup's tiles (the reference lags), in jumps, and fall; V scales on both sides of 16, from which on a tile takes
its maximum as it is because p times the scale is rounded to fp16.  Against the fp64 oracle on the same bytes."""
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
