"""The search of Alg. 2 where its kernels change: item lengths at the edges of the register classes and of the
many-workgroup form, weights that crowd one histogram bucket (ties, one value, a narrow band), weights so small that
every unit falls into the lowest buckets, tables with fewer tiers, unaligned items, maps that no search makes.  The
oracle's search runs with its threshold form of the per-unit step (`classify`): ties are the point of some cases, and the
printed form decides them by rounding."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_parity import B

pytestmark = pytest.mark.gpu


def _weights(rng, kind, shape):
    w = np.exp(rng.normal(0, 1.5, shape))
    if kind == "narrow":
        w = 1.0 + 1e-5 * rng.random(shape)
    elif kind == "one":
        w = np.full(shape, 0.37)
    elif kind == "tiny":
        w = w * 1e-38
    elif kind == "wide":
        w = np.exp(rng.normal(0, 25.0, shape))
    elif kind == "zeros":
        w = np.where(rng.random(shape) < 0.9, 0.0, w)
    elif kind == "negative":
        w = np.where(rng.random(shape) < 0.5, -w, w)
    return w.astype(np.float32)


@pytest.mark.parametrize("seq_lens,kind,budgets,tiers", [
    ((1024, 1023, 1025, 4093, 4096), "normal", (0.4, 1.0, 2.0, 4.0, 9.0), O.TIERS),
    ((4097, 16384, 16383), "normal", (0.7, 3.0, 0.05), O.TIERS),
    ((16385, 32768, 5), "normal", (0.4, 2.0, 2.0), O.TIERS),
    ((32769, 33000, 7), "normal", (0.4, 2.0, 16.0), O.TIERS),
    ((70001,), "normal", (1.0,), O.TIERS),
    ((3000, 20000), "narrow", (0.5, 3.0), O.TIERS),
    ((40000,), "narrow", (0.5,), O.TIERS),
    ((30000, 9), "one", (0.5, 3.0), O.TIERS),
    ((50000,), "one", (0.5,), O.TIERS),
    ((5000, 40000), "tiny", (1.0, 1.0), O.TIERS),
    ((5000, 30000), "tiny", (1.0, 1.0), O.TIERS),
    ((5000, 20000), "wide", (1.0, 0.3), O.TIERS),
    ((40000, 3), "wide", (1.0, 0.3), O.TIERS),
    ((5000, 20000), "zeros", (1.0, 0.05), O.TIERS),
    ((5000,), "negative", (1.0,), O.TIERS),
    ((5000, 36000), "normal", (2.0, 2.0), (0, 4, 16)),
    ((5000,), "normal", (4.5,), (2, 4, 8, 16)),
    ((300,), "normal", (8.0,), (8,)),
])
def test_allocate_at_the_edges(seq_lens, kind, budgets, tiers, monkeypatch):
    monkeypatch.setattr(O, "argmin_bits", lambda w, lam, tiers, eps: O.classify(w, lam, *O.hull_thresholds(tiers, eps)))
    print(f"[case] {seq_lens} {kind} {budgets} {tiers}", flush=True)
    b, hkv = B(), 2
    rng = np.random.default_rng(len(kind) + sum(seq_lens))
    table = [O.EPS_V_LLAMA31_8B[list(O.TIERS).index(t)] for t in tiers]
    w = [_weights(rng, kind, (hkv, T)) for T in seq_lens]
    cfg = b.Config(seq_lens, 2 * hkv, hkv, budget_bits=budgets, tiers=tiers, eps_v=[np.float32(x) for x in table])
    flat = torch.from_numpy(np.concatenate([x.reshape(-1) for x in w]))
    bits, _, lam, iters = b.rdkv_allocate_info(cfg, flat.cuda())
    bits, lam, iters = bits.cpu().numpy(), lam.cpu().numpy()[0], iters.cpu().numpy()[0]
    off = item = 0
    for s, T in enumerate(seq_lens):
        for h in range(hkv):
            ref, info = O.mckp_bisect(w[s][h], np.float32(budgets[s]), tiers, table, return_info=True)
            np.testing.assert_array_equal(bits[off:off + T], ref)
            assert iters[item] == info["iters"]
            assert np.isnan(lam[item]) if info["lam"] is None else lam[item] == info["lam"]
            off += T
            item += 1


@pytest.mark.parametrize("T", [3000, 20000, 60000])
@pytest.mark.parametrize("step", [3, 5])
@pytest.mark.parametrize("off", [-40, -1, 0, 1, 40])
def test_final_multiplier_next_to_an_early_one(T, step, off, monkeypatch):
    """A budget within a few bits of what an early multiplier spends: that step is decided on the units themselves while
    the bracket is still wide and most units lie in it."""
    monkeypatch.setattr(O, "argmin_bits", lambda w, lam, tiers, eps: O.classify(w, lam, *O.hull_thresholds(tiers, eps)))
    print(f"[case] {T} {step} {off}", flush=True)
    b, table = B(), O.EPS_V_LLAMA31_8B
    w = np.random.default_rng(T + step).random((1, T)).astype(np.float32)
    lam = float(w.max()) * 0.5 ** step            # the step-th multiplier of a search that is within the budget so far
    spent = int(O.classify(w[0], lam, *O.hull_thresholds(O.TIERS, table)).astype(np.int64).sum())
    budget = np.float32((spent + off) / T)
    cfg = b.Config([T], 1, 1, budget_bits=[float(budget)], eps_v=[np.float32(x) for x in table], rel_tol=1e-6)
    bits, _, got, iters = b.rdkv_allocate_info(cfg, torch.from_numpy(w.reshape(-1)).cuda())
    ref, info = O.mckp_bisect(w[0], budget, O.TIERS, table, rel_tol=np.float32(1e-6), return_info=True)
    np.testing.assert_array_equal(bits.cpu().numpy(), ref)
    assert iters.cpu().numpy()[0][0] == info["iters"] and got.cpu().numpy()[0][0] == info["lam"]
