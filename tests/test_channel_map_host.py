"""The channel map as the host reads it, eight channels at a time: the words of a K row of random maps against the rule (every tier's
channels in whole words, the row to an even number of them), and every value that is no bit-width, in every place (packing refuses
a map by the same function)."""
import ctypes

import numpy as np
import pytest

from paper_2605_08317_amd import binding as b


def _words(bits):
    return b.lib.rdkv_k_row_words(bits.ctypes.data_as(ctypes.c_void_p))


@pytest.mark.parametrize("seed", range(8))
def test_row_words_of_random_maps(seed):
    rng = np.random.default_rng(seed)
    for _ in range(50):
        bits = rng.choice(np.array([0, 2, 4, 8, 16], np.uint8), size=128, p=rng.dirichlet(np.full(5, 0.5)))
        words = 0
        for w, pad in ((16, 4), (8, 4), (4, 8), (2, 16)):      # slots of a tier: whole words, whole steps of four
            n = int((bits == w).sum())
            words += (n + pad - 1) // pad * pad * w // 32
        assert _words(bits) == words + words % 2


def test_values_that_are_no_width():
    rng = np.random.default_rng(0)
    maps = [rng.choice(np.array([0, 2, 4, 8, 16], np.uint8), size=128), np.zeros(128, np.uint8), np.full(128, 16, np.uint8)]
    for good in maps:
        assert _words(good) > 0 or not good.any()
        for v in set(range(256)) - {0, 2, 4, 8, 16}:
            for c in range(128):
                bits = good.copy()
                bits[c] = v
                assert _words(bits) == -1, (v, c)
