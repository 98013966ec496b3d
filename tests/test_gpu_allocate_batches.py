"""The search over batches of more items than its many-workgroup form takes at once: the scratch stays bounded whatever the
batch, and long and short items, in any order, get the maps they get alone."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_parity import B

pytestmark = pytest.mark.gpu

# sequences of 8 heads: (lengths, what they are)
BATCHES = [
    ([300] * 200 + [40000] + [300] * 311, "one long sequence among 511 short ones"),
    ([33000, 40] * 33, "528 items, half of them long"),
    ([32769] * 65, "520 items, all long: a second group of 8"),
    ([32768] * 64 + [32769], "one sequence on either side of the limit"),
]


@pytest.mark.parametrize("seq_lens,what", BATCHES, ids=[w for _, w in BATCHES])
def test_scratch_is_bounded_and_maps_are_those_of_the_items(seq_lens, what):
    b, hkv = B(), 8
    print(f"[case] {what}", flush=True)
    rng = np.random.default_rng(len(seq_lens))
    w = [np.exp(rng.normal(0, 2.0, (hkv, T))).astype(np.float32) for T in seq_lens]
    budgets = [float(x) for x in rng.choice([0.5, 1.0, 2.0, 4.0], size=len(seq_lens))]
    live, peak = {}, [0]

    @b._ALLOC_FN
    def alloc(nbytes, user):
        p = torch.cuda.caching_allocator_alloc(nbytes)
        live[p] = nbytes
        peak[0] = max(peak[0], sum(live.values()))
        return p

    @b._FREE_FN
    def free(ptr, user):
        del live[ptr]
        torch.cuda.caching_allocator_delete(ptr)

    cfg = b.Config(seq_lens, hkv, hkv, budget_bits=budgets, alloc=alloc, free_=free)
    flat = torch.from_numpy(np.concatenate([x.reshape(-1) for x in w])).cuda()
    bits, _, lam, iters = b.rdkv_allocate_info(cfg, flat)
    bits, lam, iters = bits.cpu().numpy(), lam.cpu().numpy()[0], iters.cpu().numpy()[0]
    assert not live and peak[0] < 72 << 20, f"{peak[0] >> 20} MB of scratch"
    at, sample = 0, {0, 1, len(seq_lens) // 2, len(seq_lens) - 1, int(np.argmax(seq_lens))}
    for s, T in enumerate(seq_lens):
        for h in range(hkv):
            got, item = bits[at:at + T], s * hkv + h
            at += T
            assert got.astype(np.int64).sum() <= int(np.float32(budgets[s]).astype(np.float64) * T)
            if s in sample and h in (0, hkv - 1):
                ref, info = O.mckp_bisect(w[s][h], np.float32(budgets[s]), return_info=True)
                np.testing.assert_array_equal(got, ref)
                assert iters[item] == info["iters"] and lam[item] == info["lam"]
