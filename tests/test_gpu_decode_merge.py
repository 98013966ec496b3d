"""The merging workgroups of small decode launches: slots per item on both sides of a batch of loads, every number of merging
workgroups per item (which follows the number of items and of query heads), channel-wise keys, both sides of the line between a launch
that looks and one that counts, and a workspace that every step leaves as it found it."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from paper_2605_08317_amd import workloads as W

pytestmark = pytest.mark.gpu


def _check(b, seq_lens, hkv, g, widths, mixed=False, few=None):
    wl = W.scaled(W.CONFIGS["tiny"], batch=len(seq_lens), seq_lens=tuple(seq_lens), hq=g * hkv, hkv=hkv)
    inp = W.make_inputs(wl, device="cpu")
    rng = np.random.default_rng(sum(seq_lens) + g)
    bits = [rng.choice(np.asarray(widths, np.uint8), size=(hkv, T)) for T in seq_lens]
    bits_ch = [rng.choice(np.asarray([2, 4], np.uint8), size=(hkv, 128)) for _ in seq_lens] if mixed else None
    flat = lambda m: torch.from_numpy(np.concatenate([x.reshape(-1) for x in m])).cuda()
    cfg = b.Config(seq_lens, wl.hq, hkv, budget_bits=[2.0] * len(seq_lens), s_obs=wl.s_obs,
                   k_mode=b.RDKV_K_CHANNELWISE if mixed else b.RDKV_K_TOKENWISE)
    cache = b.rdkv_pack(cfg, inp["K"].cuda(), inp["V"].cuda(), flat(bits), flat(bits_ch) if mixed else None)
    chunks = cache.stats()["n_chunks"]
    print(f"[case] {len(seq_lens)} x {hkv} items, g {g}, {chunks} chunks", flush=True)
    assert few is None or (chunks <= 256) == few
    # two queries in turn: what a step left behind would be the other query's partials
    qs = [inp["q"].cuda(), -inp["q"].cuda()]
    want = [b.rdkv_decode_attn(cache, q) for q in qs]
    for _ in range(3):
        for q, (out, lse) in zip(qs, want):
            again, again_lse = b.rdkv_decode_attn(cache, q)
            assert torch.equal(again, out) and torch.equal(again_lse, lse)
    split = lambda x: [y.float().numpy() for y in W.split_sequences(x, seq_lens, hkv, 128)]
    build = O.build_cache_mixed if mixed else O.build_cache_tokenwise
    ref = build(split(inp["K"]), split(inp["V"]), bits, *([bits_ch] if mixed else []))
    for q, (out, lse) in zip(qs, want):
        ref_out, ref_lse = O.decode(ref, q.cpu().float().numpy())
        err = np.abs(out.cpu().numpy() - ref_out).max(-1) / np.abs(ref_out).max(-1)
        assert err.max() <= 2e-3          # as in the other decode tests: fp16 products of probability and scale
        np.testing.assert_allclose(lse.cpu().numpy(), ref_lse, rtol=1e-4, atol=1e-4)
    cache.free()


@pytest.mark.parametrize("T", [513, 4096, 4097, 8449, 30000, 150001])
@pytest.mark.parametrize("g", [1, 4, 8])
def test_slots_of_one_item(T, g):
    from paper_2605_08317_amd import binding as b
    _check(b, [T], 1, g, [2])


# two chunks per item, 8, 9, 32, 33, 64, 65, 128 and 129 items among them: the last number whose launch looks and the first whose
# launch counts for 8, 4, 2 and 1 query heads per KV head
@pytest.mark.parametrize("batch,hkv,few", [(1, 3, True), (1, 8, True), (9, 1, True), (2, 8, True), (4, 8, True), (17, 2, True),
                                           (33, 1, True), (8, 8, True), (13, 5, True), (9, 8, True), (25, 4, True), (16, 8, True),
                                           (43, 3, False)])
@pytest.mark.parametrize("g", [1, 2, 4, 8])
def test_numbers_of_items(batch, hkv, few, g):
    from paper_2605_08317_amd import binding as b
    _check(b, [700 - 3 * s for s in range(batch)], hkv, g, [8, 2], few=few)


@pytest.mark.parametrize("T", [600, 9001])
@pytest.mark.parametrize("g", [2, 4])
def test_channelwise(T, g):
    from paper_2605_08317_amd import binding as b
    _check(b, [T], 2, g, [8, 4, 2, 0], mixed=True)


# more chunks than the chip has places: merging workgroups behind them (the last two), arrivals counted
@pytest.mark.parametrize("batch,hkv,g,T", [(33, 8, 4, 300), (13, 8, 4, 1100), (16, 8, 1, 1100), (12, 8, 1, 300)])
def test_channelwise_with_many_items(batch, hkv, g, T):
    from paper_2605_08317_amd import binding as b
    _check(b, [T - s for s in range(batch)], hkv, g, [8, 4, 2], mixed=True, few=False)


# one and two tiles per SIMD, as many chunks as a launch that looks has beside room for a tail, a launch that counts, tiers that
# all end in a remainder
@pytest.mark.parametrize("seq_lens,hkv,widths,few", [
    ((257,), 1, [2], True), ((512, 65), 2, [8], True), ((30600, 30600), 2, [2], True), ((61400,), 2, [4], True),
    ((5000, 70, 12001), 8, [8, 4, 2], True), ((20000, 1), 4, [16, 8, 4, 2], True), ((3000,) * 12, 8, [8, 2], False)])
@pytest.mark.parametrize("g", [1, 4, 8])
def test_rows_per_chunk(seq_lens, hkv, widths, few, g):
    from paper_2605_08317_amd import binding as b
    _check(b, list(seq_lens), hkv, g, widths, few=few)


# Merging workgroups that do not wait: whatever they find incomplete they leave to the wavefronts that store the partials.  Bits
# and workspace are those of a launch whose merging workgroups wait, whoever merges (two queries in turn: a word that was not
# put back would be the other query's).
@pytest.mark.parametrize("seq_lens,hkv,g,widths,mixed", [
    ((600,), 2, 4, [2], False), ((4097,), 1, 8, [2], False), ((30000,), 1, 4, [2], False), ((30600, 30600), 2, 4, [2], False),
    ((150001,), 1, 1, [2], False), ((150001,), 1, 8, [8, 2], False), ((700,) * 16, 4, 2, [8, 2], False), ((700,) * 4, 2, 8, [8, 2], False),
    ((3000, 20000), 4, 4, [16, 8, 4, 2], False), ((600, 9001), 2, 4, [8, 4, 2], True), ((700,) * 8, 4, 4, [8, 4, 2], True)])
@pytest.mark.parametrize("looks", [0, 3])
def test_merging_workgroups_that_give_up(seq_lens, hkv, g, widths, mixed, looks):
    from paper_2605_08317_amd import binding as b
    wl = W.scaled(W.CONFIGS["tiny"], batch=len(seq_lens), seq_lens=tuple(seq_lens), hq=g * hkv, hkv=hkv)
    inp = W.make_inputs(wl, device="cpu")
    rng = np.random.default_rng(sum(seq_lens) + g)
    bits = torch.from_numpy(rng.choice(np.asarray(widths, np.uint8), size=sum(seq_lens) * hkv)).cuda()
    bits_ch = torch.from_numpy(rng.choice(np.asarray([2, 4], np.uint8), size=len(seq_lens) * hkv * 128)).cuda() if mixed else None
    cfg = b.Config(seq_lens, wl.hq, hkv, budget_bits=[2.0] * len(seq_lens), s_obs=wl.s_obs,
                   k_mode=b.RDKV_K_CHANNELWISE if mixed else b.RDKV_K_TOKENWISE)
    cache = b.rdkv_pack(cfg, inp["K"].cuda(), inp["V"].cuda(), bits, bits_ch)
    print(f"[case] {len(seq_lens)} x {hkv} items, g {g}, looks {looks}, {cache.stats()['n_chunks']} chunks", flush=True)
    assert mixed or cache.stats()["n_chunks"] <= 256
    qs = [inp["q"].cuda(), -inp["q"].cuda()]
    set_looks = b.lib.rdkv_cache_set_looks
    set_looks.argtypes, set_looks.restype = [ctypes.c_void_p, ctypes.c_int32], None
    want = [b.rdkv_decode_attn(cache, q) for q in qs]
    assert not torch.equal(want[0][0], want[1][0])
    for n in (looks, looks, 256):
        set_looks(cache.h, n)
        for _ in range(3):
            for q, (out, lse) in zip(qs, want):
                again, again_lse = b.rdkv_decode_attn(cache, q)
                assert torch.equal(again, out) and torch.equal(again_lse, lse)
    cache.free()
