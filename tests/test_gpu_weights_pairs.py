"""Token weights of short items, whose key tiles have a workgroup each or one for two, on both sides of the lines: 34 and 35 tiles (a
workgroup each and 34 runs; pairs), 66 and 67 (34 runs of pairs; a launch for the log-sum-exp), 512 and 513 tiles in all, items that
start in the middle of a pair.  Against the oracle, and the same bits with channel weights."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_parity import B, WEIGHT_RTOL, _np, _split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles,others", [(33, ()), (34, (64,)), (35, (65, 700)), (36, (2300, 65)), (65, (65, 65)), (66, (65, 4224)), (67, (70,)),
                                          (64, (4096,) * 3), (64, (4096, 4096, 4097))])
@pytest.mark.parametrize("hq,s_obs", [(2, 32), (4, 64), (8, 33)])
def test_runs_of_one_tile_and_two(tiles, others, hq, s_obs):
    lens, hkv, d = (64 * tiles - 3, *others), 2, 128
    print(f"[case] {lens} hq {hq} s_obs {s_obs}", flush=True)
    b, gen = B(), torch.Generator().manual_seed(tiles + hq)
    K = torch.randn(sum(lens) * hkv * d, generator=gen).to(torch.bfloat16)
    Q = torch.randn((len(lens), hq, s_obs, d), generator=gen).to(torch.bfloat16)
    cfg = b.Config(lens, hq, hkv, s_obs=s_obs, pool_kernel=5)
    w, _ = b.rdkv_weights(cfg, K.cuda(), Q.cuda())
    assert torch.equal(w, b.rdkv_weights(cfg, K.cuda(), Q.cuda(), want_channel=True)[0])
    w = w.cpu().numpy().astype(np.float64)
    off = 0
    for s, (T, Ks) in enumerate(zip(lens, _split(K, lens, hkv, d))):
        ref = O.avg_pool(O.token_weights(Ks, _np(Q[s])), 5)
        got = w[off:off + hkv * T].reshape(hkv, T)
        off += hkv * T
        assert (np.abs(got - ref) / (np.abs(ref) + 1e-6 * ref.max())).max() <= WEIGHT_RTOL
