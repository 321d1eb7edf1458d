"""The order of a step's work items: the dearest first and equal ones in their
groups' order, for short lists and for those that are sorted by counting."""
import numpy as np
import pytest

from paper_1603_06958_amd import inputs
from workdump import dry_run


@pytest.mark.parametrize("k,lo,hi", [(40, 10, 300), (3000, 100, 110), (9000, 20, 900), (2500, 60, 60), (3000, 0, 2500)])
def test_dearest_items_first(k, lo, hi):
    d, _ = dry_run(inputs.random_family(k, lo, hi, seed=k), cols_per_item=64)
    g, it, r, cm = d["groups"], d["items"], d["ranges"][0], d["colmap"]
    assert len(d["steps"]) == 1  # the whole family: columns are the length order's positions
    pref = np.concatenate([[0], np.cumsum(d["len"][cm].astype(np.int64))])
    lpr = np.maximum(g["lpr"], 1)
    dwords = ((g["W"] + lpr - 1) // lpr).astype(np.int64)
    counted = 0
    for c in range(4):
        x = it[r["begin"][c]:r["end"][c]]
        counted += len(x) >= 1024
        cost = dwords[x["group"]] * (pref[x["c1"]] - pref[x["c0"]])
        key = np.stack([-cost, -dwords[x["group"]], x["group"].astype(np.int64), x["c0"].astype(np.int64)])
        order = np.lexsort(key[::-1])  # by cost, then as they were cut: widest groups first, each from its first column
        assert np.array_equal(order, np.arange(len(x)))
    assert (counted > 0) == (k > 40)
