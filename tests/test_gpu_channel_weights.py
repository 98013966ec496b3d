"""Channel weights from the workgroups behind the second pass's (items of up to 34 runs) and from the launch of the log-sum-exp, for
every form of the passes, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_parity import B, _np, _split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,s_obs", [(2, 32), (4, 64), (8, 33)])      # 32, 128 and 132 rows an item
@pytest.mark.parametrize("lens", [(33,), (64, 2000, 100), (34 * 64,), (66 * 64, 64), (67 * 64,), (35 * 64, 65), tuple(40 + 13 * k for k in range(40))])
def test_channel_weights_of_few_runs_and_many(lens, hq, s_obs):
    hkv, d = 2, 128
    if min(lens) < s_obs:
        lens = tuple(T + s_obs for T in lens)
    print(f"[case] {lens[:4]} hq {hq} s_obs {s_obs}", flush=True)
    b, gen = B(), torch.Generator().manual_seed(len(lens) + hq)
    K = torch.randn(sum(lens) * hkv * d, generator=gen).to(torch.bfloat16)
    Q = torch.randn((len(lens), hq, s_obs, d), generator=gen).to(torch.bfloat16)
    w_ch = b.rdkv_weights(b.Config(lens, hq, hkv, s_obs=s_obs), K.cuda(), Q.cuda(), want_channel=True)[1].cpu().numpy().reshape(-1, d)
    for s, Ks in enumerate(_split(K, lens, hkv, d)):
        np.testing.assert_allclose(w_ch[s * hkv:(s + 1) * hkv], O.channel_weights(Ks, _np(Q[s])), rtol=1e-5)


# Items of few runs whose channel weights the launch of the log-sum-exp makes all the same (more than 128 of up to 64 rows, than 256 of up to
# 128): 128, 130, 256 and 258 items, and the same token weights as without.
@pytest.mark.parametrize("hq,s_obs", [(2, 32), (4, 64), (8, 33)])
@pytest.mark.parametrize("seqs", [64, 65, 128, 129])
def test_channel_weights_of_many_items(seqs, hq, s_obs):
    hkv, d, lens = 2, 128, [64 + k % 3 for k in range(seqs)]
    print(f"[case] {seqs} sequences hq {hq} s_obs {s_obs}", flush=True)
    b, gen = B(), torch.Generator().manual_seed(seqs + hq)
    K = torch.randn(sum(lens) * hkv * d, generator=gen).to(torch.bfloat16)
    Q = torch.randn((seqs, hq, s_obs, d), generator=gen).to(torch.bfloat16)
    cfg = b.Config(lens, hq, hkv, s_obs=s_obs, budget_bits=[2.0] * seqs)
    w, w_ch = b.rdkv_weights(cfg, K.cuda(), Q.cuda(), want_channel=True)
    assert torch.equal(w, b.rdkv_weights(cfg, K.cuda(), Q.cuda())[0])
    w_ch = w_ch.cpu().numpy().reshape(-1, d)
    for s, Ks in enumerate(_split(K, lens, hkv, d)):
        np.testing.assert_allclose(w_ch[s * hkv:(s + 1) * hkv], O.channel_weights(Ks, _np(Q[s])), rtol=1e-5)
