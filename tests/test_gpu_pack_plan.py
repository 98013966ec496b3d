"""The tables that the launch with the position lists makes for the packing kernels: one to 300 items (a wavefront per item
down to one thread, a round of them and more), items without tokens, of one block of the bit map and of several."""
import numpy as np
import pytest

from test_gpu_mixed import _assert_cache_equal_mixed, _pack_both_mixed
from test_gpu_parity import B, _assert_cache_equal, _inputs, _pack_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seqs", [1, 3, 17, 65, 128, 150])
@pytest.mark.parametrize("mode", ["token", "groups", "channel"])
def test_plan(seqs, mode):
    b, rng = B(), np.random.default_rng(seqs)
    lens = [int(x) for x in rng.integers(0, 70, seqs)]
    lens[seqs // 2] = 2100
    wl, inp, dev = _inputs("tiny", batch=seqs, budgets=(2.0,) * seqs, seq_lens=tuple(lens))
    tiers = np.array([0, 2, 4, 8, 16], np.uint8)
    bits = [rng.choice(tiers, size=(wl.hkv, T), p=rng.dirichlet(np.ones(5))) for T in lens]
    if mode == "token":
        cache, ref = _pack_both(b, wl, inp, dev, bits)
        _assert_cache_equal(b, cache, ref)
    else:
        bc = [rng.choice(tiers, size=(wl.hkv, 128), p=rng.dirichlet(np.ones(5))) for _ in lens]
        cache, ref = _pack_both_mixed(b, wl, inp, dev, bits, bc, per_channel_scale=mode == "channel")
        _assert_cache_equal_mixed(b, cache, ref)
    cache.free()
