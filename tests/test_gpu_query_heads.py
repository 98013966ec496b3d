"""A query head with values that are not finite, or too large for the scaled fp16 operand, is that head's affair: the other
heads of its KV head share matrix products with it and must come out bit for bit as beside a finite head, in every form of
the decode step."""
import numpy as np
import pytest
import torch

from paper_2605_08317_amd import workloads as W
from test_gpu_parity import B

pytestmark = pytest.mark.gpu


def _decode(b, form, wl, dev):
    """A function of the query that runs one form of the decode step."""
    T = wl.seq_lens[0]
    if form == "bf16":
        return lambda q: b.rdkv_decode_attn_bf16(dev["K"], dev["V"], [T], wl.hq, wl.hkv, q)
    rng = np.random.default_rng(T)
    mixed = form.startswith("channel")
    widths = [16, 8, 4, 2, 0]
    cfg = b.Config([T], wl.hq, wl.hkv, k_mode=b.RDKV_K_CHANNELWISE if mixed else b.RDKV_K_TOKENWISE,
                   k_scale_per_channel=int(form == "channel, one scale"))
    bits = torch.from_numpy(rng.choice(np.asarray(widths, np.uint8), size=wl.hkv * T)).cuda()
    bits_ch = torch.from_numpy(rng.choice(np.asarray(widths, np.uint8), size=wl.hkv * 128)).cuda() if mixed else None
    cache = b.rdkv_pack(cfg, dev["K"], dev["V"], bits, bits_ch)
    if form == "tail":
        b.rdkv_cache_reserve_tail(cache, 80)
        new = torch.randn((80, 1, wl.hkv, 128), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16).cuda()
        for i in range(80):
            b.rdkv_cache_append(cache, new[i], new[79 - i])
    return lambda q: b.rdkv_decode_attn(cache, q)


@pytest.mark.parametrize("g", [2, 4, 8])
@pytest.mark.parametrize("form,T", [("token", 1500), ("token", 100000),     # 16-bit rows along, and in a launch of their own
                                    ("tail", 300), ("channel", 1500), ("channel, one scale", 1500), ("bf16", 3000)])
def test_other_heads_do_not_see_it(form, T, g):
    b = B()
    print(f"[case] {form} T {T} g {g}", flush=True)
    wl = W.scaled(W.CONFIGS["tiny"], seq_lens=(T,), hq=2 * g, hkv=2)
    dev = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in W.make_inputs(wl, device="cpu").items()}
    step = _decode(b, form, wl, dev)
    out, lse = step(dev["q"])
    assert torch.isfinite(out).all()
    for k, value in enumerate((float("nan"), float("inf"), -float("inf"), 3.0e5)):
        head = (1 + 3 * k) % g + g * (k & 1)
        q = dev["q"].clone()
        q[0, head, 5 * k] = value
        got, got_lse = step(q)
        others = [h for h in range(wl.hq) if h != head]
        assert torch.equal(got[:, others], out[:, others]), f"{value} in head {head} reached another head"
        assert torch.equal(got_lse[:, others], lse[:, others])
