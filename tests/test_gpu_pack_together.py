"""Channel-wise packing on both sides of the line between one launch for K and V and one for each (4096 workgroups: 64 items whose
longest has 21 tiles, 22 tiles), in both K formats: the arena must equal the oracle's byte for byte."""
import numpy as np
import pytest

from test_gpu_mixed import _assert_cache_equal_mixed, _pack_both_mixed
from test_gpu_parity import B, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("tiles", [21, 22])
def test_one_launch_and_two(tiles, per_channel):
    b, rng = B(), np.random.default_rng(tiles)
    lens = (64 * tiles - 5,) + tuple(int(x) for x in rng.integers(1, 200, 31))
    wl, inp, dev = _inputs("tiny", batch=32, seq_lens=lens)
    assert wl.hkv == 2
    tiers = np.array([0, 2, 4, 8, 16], np.uint8)
    bt = [np.full((2, lens[0]), 4, np.uint8)] + [rng.choice(tiers, size=(2, T)) for T in lens[1:]]
    bc = [rng.choice(tiers, size=(2, 128), p=[.1, .4, .3, .15, .05]) for _ in lens]
    cache, ref = _pack_both_mixed(b, wl, inp, dev, bt, bc, per_channel)
    _assert_cache_equal_mixed(b, cache, ref)
    cache.free()
