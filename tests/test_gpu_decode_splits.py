"""Decode over items of one, few and many partials: the finish of a single chunk, the merge's slot groups at every number
of query heads per KV head, more slots than one round of its loads."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from paper_2605_08317_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [1, 2, 4, 8])
@pytest.mark.parametrize("T,widths", [(1, [8]), (50, [2]), (257, [4]), (700, [16, 8, 4, 2]), (3001, [8, 4, 2, 0]), (24000, [2])])
@pytest.mark.parametrize("hkv", [1, 2])
def test_partials_of_an_item(g, T, widths, hkv):
    from paper_2605_08317_amd import binding as b
    print(f"[case] g {g} T {T} widths {widths} hkv {hkv}", flush=True)
    wl = W.scaled(W.CONFIGS["tiny"], seq_lens=(T,), hq=g * hkv, hkv=hkv)
    inp = W.make_inputs(wl, device="cpu")
    rng = np.random.default_rng(T + g)
    bits = rng.choice(np.asarray(widths, np.uint8), size=(hkv, T))
    cfg = b.Config([T], wl.hq, wl.hkv, budget_bits=[2.0], s_obs=wl.s_obs)
    cache = b.rdkv_pack(cfg, inp["K"].cuda(), inp["V"].cuda(), torch.from_numpy(bits.reshape(-1)).cuda())
    out, lse = b.rdkv_decode_attn(cache, inp["q"].cuda())
    again, _ = b.rdkv_decode_attn(cache, inp["q"].cuda())
    torch.cuda.synchronize()
    ref = O.build_cache_tokenwise([x.float().numpy() for x in W.split_sequences(inp["K"], [T], hkv, 128)],
                                  [x.float().numpy() for x in W.split_sequences(inp["V"], [T], hkv, 128)], [bits])
    ref_out, ref_lse = O.decode(ref, inp["q"].float().numpy())
    out, lse = out.cpu().numpy(), lse.cpu().numpy()
    err = np.abs(out - ref_out).max(-1) / np.abs(ref_out).max(-1)
    assert err.max() <= 2e-3
    np.testing.assert_allclose(lse, ref_lse, rtol=1e-4, atol=1e-4)
    assert np.array_equal(again.cpu().numpy(), out)
    cache.free()
