"""Channel-wise decode over K rows of every shape of a tile's loads: whole runs of four words, a run of two at the end (whose
lanes read past their own words), rows at both ends of a kernel's range, steps up to 32 and beyond, both K formats; V tiles of every
width; fewer tiles than wavefronts, one more, and several per wavefront.  Against the fp64 oracle on the same bytes."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from test_gpu_mixed import _pack_both_mixed
from test_gpu_parity import B, _check_decode, _inputs, _np

pytestmark = pytest.mark.gpu

# channels of 16, 8, 4, 2 bits -> words of a row
ROWS = [(0, 0, 0, 32), (0, 0, 0, 96), (0, 0, 80, 0), (0, 0, 37, 91), (0, 0, 112, 0), (0, 4, 120, 4), (0, 72, 0, 0), (0, 120, 8, 0),
        (68, 0, 0, 60), (124, 0, 0, 0), (125, 1, 1, 1)]


@pytest.mark.parametrize("per_channel", [False, True])
@pytest.mark.parametrize("g", [4, 8])
@pytest.mark.parametrize("row", ROWS)
def test_rows(row, g, per_channel):
    print(f"[case] row {row} g {g} per_channel {per_channel}", flush=True)
    b, rng = B(), np.random.default_rng(sum(row) + g)
    wl, inp, dev = _inputs("batch70b", batch=3, len_range=(60, 2300), hq=2 * g, hkv=2)
    bt = [rng.choice(np.array([0, 2, 4, 8, 16], np.uint8), size=(2, T), p=[.1, .3, .3, .2, .1]) for T in inp["seq_lens"]]
    widths = np.repeat(np.array([16, 8, 4, 2, 0], np.uint8), [*row, 128 - sum(row)])
    bc = [np.stack([rng.permutation(widths) for _ in range(2)]) for _ in inp["seq_lens"]]
    cache, ref = _pack_both_mixed(b, wl, inp, dev, bt, bc, per_channel)
    out, lse = b.rdkv_decode_attn(cache, dev["q"])
    torch.cuda.synchronize()
    ref_out, ref_lse = O.decode(ref, _np(inp["q"]))
    _check_decode(out, lse, ref_out, ref_lse)
    cache.free()
