"""The steps of the search that the histogram leaves: on all units (up to 8K, up to 16K in a launch of at most 64 items, then on a
list) and, where they are listed, on up to 64, 256, 512, 1024 and more open units, three at a time up to 1024.  A band of weights
too narrow for the histogram straddles the threshold, so that every item has more such steps than a round or a first group of them
takes.  Against the oracle's search: maps, multipliers and step counts."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_parity import B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_seqs", [2, 32, 33])
@pytest.mark.parametrize("T", [4096, 4097, 8192, 8193, 16384, 16385, 33000])
@pytest.mark.parametrize("band", [40, 64, 65, 256, 257, 512, 513, 1024, 1025])
def test_steps_on_a_band(n_seqs, T, band, monkeypatch):
    monkeypatch.setattr(O, "argmin_bits", lambda w, lam, tiers, eps: O.classify(w, lam, *O.hull_thresholds(tiers, eps)))
    print(f"[case] {n_seqs} sequences, the first of {T}, band of {band}", flush=True)
    b, hkv, table, tiers = B(), 2, [O.EPS_V_LLAMA31_8B[list(O.TIERS).index(t)] for t in (0, 16)], (0, 16)
    rng = np.random.default_rng(T + band)
    lens = [T] + [5 + s for s in range(n_seqs - 1)]
    w = [np.exp(rng.normal(0, 1.0, (hkv, n))).astype(np.float32) for n in lens]
    above = T // 5
    for h in range(hkv):                  # `above` units over the band, the others below it
        x = np.sort(w[0][h])[::-1]
        x[:above] = 1.5 + x[:above]
        x[above:] *= 0.9 / x[above]
        x[above:above + band] = (1.0 + 1e-4 * rng.random(band)).astype(np.float32)
        w[0][h] = rng.permutation(x)
    budgets = [16.0 * (above + band * 0.37) / T] + [2.0] * (n_seqs - 1)
    cfg = b.Config(lens, 2 * hkv, hkv, budget_bits=budgets, tiers=tiers, eps_v=[np.float32(x) for x in table], rel_tol=1e-6)
    flat = torch.from_numpy(np.concatenate([x.reshape(-1) for x in w]))
    bits, _, lam, iters = b.rdkv_allocate_info(cfg, flat.cuda())
    bits, lam, iters = bits.cpu().numpy(), lam.cpu().numpy()[0], iters.cpu().numpy()[0]
    off = item = 0
    for s in range(2):
        for h in range(hkv):
            ref, info = O.mckp_bisect(w[s][h], np.float32(budgets[s]), tiers, table, rel_tol=np.float32(1e-6), return_info=True)
            np.testing.assert_array_equal(bits[off:off + lens[s]], ref)
            assert iters[item] == info["iters"]
            assert np.isnan(lam[item]) if info["lam"] is None else lam[item] == info["lam"]
            assert s or info["iters"] >= 13
            off += lens[s]
            item += 1
