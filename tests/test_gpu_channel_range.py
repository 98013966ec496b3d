"""One scale per key channel: the smallest and the largest number of every channel over the kept rows, at row counts around a
wavefront's load, a workgroup's and the whole launch's, with the extremes in the first and the last kept row and numbers of one
sign and of both, and zeros."""
import numpy as np
import pytest
import torch

from test_gpu_mixed import _assert_cache_equal_mixed, _pack_both_mixed
from test_gpu_parity import B, _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sign", ["both", "positive", "negative", "zeros"])
@pytest.mark.parametrize("T,kept", [(1, 1), (70, 5), (300, 255), (300, 256), (300, 257), (1200, 1025), (34000, 33025)])
def test_range_of_a_channel(T, kept, sign):
    if T > 30000 and sign != "both":
        pytest.skip("the largest once")
    b = B()
    wl, inp, dev = _inputs("tiny", seq_lens=(T,), hq=2, hkv=2)
    rng = np.random.default_rng(T + kept)
    bits = np.zeros((2, T), np.uint8)
    K = inp["K"].reshape(2, T, 128).clone()
    for h in range(2):
        rows = np.sort(rng.permutation(T)[:kept])
        bits[h, rows] = rng.choice(np.array([2, 4, 8, 16], np.uint8), size=kept)
        if sign == "positive":
            K[h] = K[h].abs() + 0.5
        elif sign == "negative":
            K[h] = -K[h].abs() - 0.5
        elif sign == "zeros":      # (of one sign per channel: the oracle's largest of both is whichever NumPy met first)
            K[h] = torch.where(torch.from_numpy(rng.random(128) < 0.5), 0.0, -0.0).to(K.dtype)
        else:
            K[h, rows[0]], K[h, rows[-1]] = -19.0, 21.0
    inp["K"] = K.reshape(inp["K"].shape)
    dev["K"] = inp["K"].cuda()
    print(f"[case] {kept} of {T} rows, {sign}", flush=True)
    ch = rng.choice(np.array([2, 4, 8], np.uint8), size=(2, 128))
    cache, ref = _pack_both_mixed(b, wl, inp, dev, [bits], [ch], per_channel_scale=True)
    _assert_cache_equal_mixed(b, cache, ref)
    cache.free()
