"""The pack kernels at the edges of their tiles: rows per tier one below, at and above 64, tiers without rows, and values
that take the quantizer out of its fast form (ranges beyond fp16, infinite offsets, constant groups, signed zeros,
subnormal scales).  The arena must equal the oracle's byte for byte, padding included."""
import numpy as np
import pytest
import torch

from oracle import rdkv_oracle as O
from paper_2605_08317_amd import workloads as W
from test_gpu_mixed import _pack_both_mixed
from test_gpu_parity import B, _inputs, _pack_both

pytestmark = pytest.mark.gpu


def _bits(counts, T, rng):
    x = np.zeros(T, np.uint8)
    order, at = rng.permutation(T), 0
    for b, n in zip((16, 8, 4, 2), counts):
        x[order[at:at + n]] = b
        at += n
    return x


def _odd_values(K):
    """Overwrites rows of a [hkv, T, 128] bf16 tensor with values at the ends of the format."""
    K[:, 0::7] *= 1e-7                          # subnormal fp16 scales
    K[:, 1::11, :32] = 3.0                      # constant groups
    K[:, 2::13, 32:64] = -0.0
    K[:, 3::17, 64:96] *= 3e5                   # scale and offset beyond fp16
    K[:, 4::19] = torch.where(torch.rand(K[:, 4::19].shape) < 0.5, 0.0, 1e-30).to(K.dtype)


@pytest.mark.parametrize("counts", [
    (63, 64, 65, 127), (0, 1, 0, 128), (64, 0, 0, 0), (1, 1, 1, 1), (129, 65, 0, 63), (0, 0, 0, 0), (65, 0, 191, 64)])
@pytest.mark.parametrize("mixed", [False, True])
def test_tile_edges(counts, mixed):
    b, rng = B(), np.random.default_rng(sum(counts) + mixed)
    wl, inp, dev = _inputs("tiny", seq_lens=(400,))
    bits = [np.stack([_bits(counts, 400, rng), _bits(counts[::-1], 400, rng)])]
    if mixed:
        bc = [rng.choice(np.array([0, 2, 4, 8, 16], np.uint8), size=(wl.hkv, 128), p=[.1, .4, .3, .15, .05])]
        cache, ref = _pack_both_mixed(b, wl, inp, dev, bits, bc)
    else:
        cache, ref = _pack_both(b, wl, inp, dev, bits)
    assert np.array_equal(cache.export(b.RDKV_EXPORT_ARENA, np.uint8), ref["arena"])
    cache.free()


@pytest.mark.parametrize("mixed", [False, True])
def test_values_at_the_ends_of_the_formats(mixed):
    b, rng = B(), np.random.default_rng(5)
    wl, inp, _ = _inputs("tiny", seq_lens=(600,))
    for name in ("K", "V"):
        for v in W.split_sequences(inp[name], inp["seq_lens"], wl.hkv, wl.d):
            _odd_values(v)
    dev = {k: (v.cuda() if torch.is_tensor(v) else v) for k, v in inp.items()}
    bits = [rng.choice(np.array([2, 4, 8], np.uint8), size=(wl.hkv, 600))]
    with np.errstate(all="ignore"):
        if mixed:
            bc = [rng.choice(np.array([2, 4, 8], np.uint8), size=(wl.hkv, 128))]
            cache, ref = _pack_both_mixed(b, wl, inp, dev, bits, bc)
        else:
            cache, ref = _pack_both(b, wl, inp, dev, bits)
    assert np.array_equal(cache.export(b.RDKV_EXPORT_ARENA, np.uint8), ref["arena"])
    cache.free()
