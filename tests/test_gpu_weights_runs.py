"""Token and channel weights where their kernels' partition can go wrong: window-row counts at the edges of the row
tiles and sweeps, items shorter than a key tile and runs of tiles that span several items, keys hidden by the causal
mask in a run's first tile, and logits further apart than fp32 carries around a fixed reference."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_parity import B, WEIGHT_RTOL, _np, _split

pytestmark = pytest.mark.gpu

MANY = tuple(64 + 37 * k for k in range(24))     # 48 items of 2 .. 15 tiles


@pytest.mark.parametrize("seq_lens,hq,hkv,s_obs,causal,spike", [
    ((1,), 2, 2, 1, 1, 0),
    ((63, 64, 65), 4, 4, 32, 1, 0),
    ((129, 64), 2, 1, 32, 1, 0),                 # 64 rows
    ((200, 66), 2, 1, 33, 1, 0),                 # 66 rows
    ((300,), 8, 1, 16, 0, 0),                    # 128 rows
    ((300, 1), 8, 1, 1, 1, 0),                   # a sequence of one token
    ((513,), 8, 1, 17, 1, 0),                    # 136 rows
    ((640,), 8, 1, 32, 1, 0),                    # 256 rows
    ((640, 100), 8, 1, 33, 1, 0),                # 264 rows: a second sweep
    ((1000,), 16, 2, 64, 1, 0),                  # 512 rows
    (MANY, 8, 2, 32, 1, 0),
    ((2000,), 8, 2, 64, 1, 120.0),
    ((2000, 700), 2, 2, 32, 0, 120.0),
])
def test_weights_over_row_and_tile_edges(seq_lens, hq, hkv, s_obs, causal, spike):
    print(f"[case] {seq_lens} hq {hq} hkv {hkv} s_obs {s_obs} causal {causal} spike {spike}", flush=True)
    b, d = B(), 128
    gen = torch.Generator().manual_seed(sum(seq_lens) + hq)
    K = torch.randn(sum(seq_lens) * hkv * d, generator=gen)
    Q = torch.randn((len(seq_lens), hq, s_obs, d), generator=gen)
    if spike:                                    # one key per item far above the first keys of its tile
        u = torch.randn(d, generator=gen)
        u /= u.norm()
        Q += 9.5 * u
        at = 0
        for T in seq_lens:
            K[at:at + hkv * T * d].view(hkv, T, d)[:, T // 128 * 64 + 40] += spike * u
            at += hkv * T * d
    K, Q = K.to(torch.bfloat16), Q.to(torch.bfloat16)
    cfg = b.Config(seq_lens, hq, hkv, s_obs=s_obs, pool_kernel=5, causal=causal)
    w_tok, w_ch = b.rdkv_weights(cfg, K.cuda(), Q.cuda(), want_channel=True)
    w_tok, w_ch = w_tok.cpu().numpy().astype(np.float64), w_ch.cpu().numpy().reshape(-1, d)
    off = 0
    for s, (T, Ks) in enumerate(zip(seq_lens, _split(K, seq_lens, hkv, d))):
        ref = O.avg_pool(O.token_weights(Ks, _np(Q[s]), causal=bool(causal)), 5)
        got = w_tok[off:off + hkv * T].reshape(hkv, T)
        off += hkv * T
        err = np.abs(got - ref) / (np.abs(ref) + 1e-6 * ref.max())
        # (spiked logits of 145 powers of two: the log-sum-exp is rounded to 1.5e-5 / 2 there, 5e-6 of a weight; over these
        # and other seeds and spikes of 20 to 120 at most 2.4e-6 came out, 1.3e-6 with a running maximum in every tile)
        assert err.max() <= WEIGHT_RTOL, f"sequence {s}: {err.max():.2e}"
        np.testing.assert_allclose(w_ch[s * hkv:(s + 1) * hkv], O.channel_weights(Ks, _np(Q[s])), rtol=1e-5)


# One launch fewer where items have few runs, with and without the channel weights: the same additions, so the same bits.
@pytest.mark.parametrize("seq_lens,hq,hkv,s_obs", [
    ((1,), 2, 2, 1),
    ((1920, 33, 63, 64, 65, 1025), 2, 2, 32),    # 64 rows; 30 runs, 17
    ((1024, 300), 8, 2, 32),                     # 128 rows; 16 runs
    ((1921, 896), 8, 1, 32),                     # 256 rows; 31 runs: a launch of its own
    ((1857, 896), 8, 1, 33),                     # 264 rows: a second sweep
    ((500, 80), 16, 2, 64),                      # 512 rows
    (tuple(7000 + 101 * k for k in range(8)), 8, 2, 32),      # 16 items that share 512 runs
    (tuple(1500 + 101 * k for k in range(24)), 8, 2, 64),     # 48 items, runs that span two of them
])
def test_log_sum_exp_inside_the_second_pass(seq_lens, hq, hkv, s_obs):
    print(f"[case] {seq_lens} hq {hq} hkv {hkv} s_obs {s_obs}", flush=True)
    b, d = B(), 128
    gen = torch.Generator().manual_seed(len(seq_lens) + hq)
    K = torch.randn(sum(seq_lens) * hkv * d, generator=gen).to(torch.bfloat16).cuda()
    Q = torch.randn((len(seq_lens), hq, s_obs, d), generator=gen).to(torch.bfloat16).cuda()
    cfg = b.Config(seq_lens, hq, hkv, s_obs=s_obs)
    w_tok, _ = b.rdkv_weights(cfg, K, Q)
    assert torch.equal(w_tok, b.rdkv_weights(cfg, K, Q, want_channel=True)[0])
