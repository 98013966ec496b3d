"""What a pass reads about its batch, an entry per sequence: along with the launches up to 32 sequences, a table in device memory
beyond that; one, three and eight heads (the item's sequence comes from a reciprocal), more sequences than a wavefront has lanes."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_parity import B, WEIGHT_RTOL, _np, _split

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv", [1, 3, 8])
@pytest.mark.parametrize("batch", [31, 32, 33, 65, 130])
def test_entries(batch, hkv):
    print(f"[case] {batch} sequences, {hkv} heads", flush=True)
    b, d, s_obs = B(), 128, 4
    rng, gen = np.random.default_rng(batch), torch.Generator().manual_seed(batch)
    lens = [int(x) for x in rng.integers(s_obs, 140, batch)]
    lens[batch // 2], lens[-1] = 1500, 1100       # several runs and blocks of the bit map
    K = torch.randn(sum(lens) * hkv * d, generator=gen).to(torch.bfloat16)
    Q = torch.randn((batch, hkv, s_obs, d), generator=gen).to(torch.bfloat16)
    budgets = [float(x) for x in rng.uniform(0.5, 6.0, batch).astype(np.float32)]
    cfg = b.Config(lens, hkv, hkv, budget_bits=budgets, s_obs=s_obs)
    w, _ = b.rdkv_weights(cfg, K.cuda(), Q.cuda())
    bits, _ = b.rdkv_allocate(cfg, w, None)
    w, bits = w.cpu().numpy(), bits.cpu().numpy()
    off = 0
    for s, (T, Ks) in enumerate(zip(lens, _split(K, lens, hkv, d))):
        ref = O.avg_pool(O.token_weights(Ks, _np(Q[s])), 5)
        got = w[off:off + hkv * T].reshape(hkv, T)
        err = np.abs(got.astype(np.float64) - ref) / (np.abs(ref) + 1e-6 * ref.max())
        assert err.max() <= WEIGHT_RTOL, f"sequence {s}: {err.max():.2e}"
        if s in (0, batch // 2, batch - 2, batch - 1):
            for h in range(hkv):
                np.testing.assert_array_equal(bits[off + h * T:off + (h + 1) * T], O.mckp_bisect(got[h], np.float32(budgets[s])))
        off += hkv * T
