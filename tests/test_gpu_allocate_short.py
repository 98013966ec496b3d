"""Items of up to 4K units, whose undecided steps are taken on all units: lengths around a wavefront, a block and the longest,
against weights that leave one step or all of them undecided."""
import pytest

import test_gpu_allocate_edges as edges
from oracle import rdkv_oracle as O

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["normal", "narrow", "one", "tiny", "wide", "zeros"])
@pytest.mark.parametrize("tiers", [O.TIERS, (0, 4, 16)])
def test_short_items(kind, tiers, monkeypatch):
    seq_lens, budgets = (1, 2, 63, 64, 65, 1023, 2049, 4095, 4096), (4.0, 3.0, 0.5, 1.0, 2.0, 2.0, 0.7, 1.0, 3.0)
    edges.test_allocate_at_the_edges(seq_lens, kind, budgets, tiers, monkeypatch)
