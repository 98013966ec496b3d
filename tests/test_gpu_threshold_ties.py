"""A token whose weight lies next to a threshold of its search can come out on either side of it when the weights are summed
in another order.  With channel-wise keys in groups of 32 that one token moves every later retained token of its segment to
another group, where its key is quantized against other neighbours: the head's output then changes by percents.  That is
the format's sensitivity and no error of a kernel: on either map the decode step is the oracle's on that same map."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from paper_2605_08317_amd import workloads as W
from test_gpu_full_size import _check_sampled_items
from test_gpu_mixed import _pack_both_mixed
from test_gpu_parity import B, _np, _check_decode, _inputs

pytestmark = pytest.mark.gpu


def _other_side(w, bits, lam, eps):
    """The map with the token nearest a threshold moved across it."""
    tiers, r = O.hull_thresholds(O.TIERS, eps)
    distance = np.abs(w[:, None].astype(np.float64) / (lam * np.asarray(r, np.float64)) - 1.0)
    t, k = np.unravel_index(np.argmin(distance), distance.shape)
    assert bits[t] in (tiers[k], tiers[k + 1])
    moved = bits.copy()
    moved[t] = tiers[k] if bits[t] == tiers[k + 1] else tiers[k + 1]
    return moved, float(distance[t, k])


@pytest.mark.parametrize("T", [50021])
def test_decode_on_both_sides_of_the_nearest_threshold(T):
    b = B()
    wl, inp, dev = _inputs("layer8b", seq_lens=(T,), hq=8, hkv=2)
    eps = O.EPS_V_LLAMA31_8B
    cfg = b.Config(inp["seq_lens"], wl.hq, wl.hkv, budget_bits=inp["budgets"], s_obs=wl.s_obs, k_mode=b.RDKV_K_CHANNELWISE)
    w_tok, w_ch = b.rdkv_weights(cfg, dev["K"], dev["Q_obs"], want_channel=True)
    bits_tok, bits_ch, lam, _ = b.rdkv_allocate_info(cfg, w_tok, w_ch)
    cache = b.rdkv_pack(cfg, dev["K"], dev["V"], bits_tok, bits_ch)
    own, own_lse = b.rdkv_decode_attn(cache, dev["q"])
    torch.cuda.synchronize()
    # maps, packed bytes and decode of both heads from the library's own weights
    _check_sampled_items(b, wl, inp, cache, own, own_lse, w_tok.cpu(), [(0, 0), (0, 1)], mixed=True,
                         w_ch=w_ch.cpu().numpy().reshape(-1, 128))
    cache.free()
    # and with one token of every head on the other side
    w, lam = w_tok.cpu().numpy().reshape(wl.hkv, T), lam.cpu().numpy()[0]
    bt, bc = bits_tok.cpu().numpy().reshape(wl.hkv, T), bits_ch.cpu().numpy().reshape(wl.hkv, 128)
    moved, distance = zip(*(_other_side(w[h], bt[h], lam[h], eps) for h in range(wl.hkv)))
    cache, ref = _pack_both_mixed(b, wl, inp, dev, [np.stack(moved)], [bc])
    out, lse = b.rdkv_decode_attn(cache, dev["q"])
    torch.cuda.synchronize()
    assert np.array_equal(cache.export(b.RDKV_EXPORT_ARENA, np.uint8), ref["arena"])
    _check_decode(out, lse, *O.decode(ref, _np(inp["q"])))
    for h in range(wl.hkv):
        x, y = (t[0, h * 4:h * 4 + 4].double() for t in (out, own))
        print(f"[tie] head {h}: a weight {distance[h]:.1e} from its threshold moved across it changes the output by "
              f"{((x - y).norm() / y.norm()).item():.1e}", flush=True)
    cache.free()
