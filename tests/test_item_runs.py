"""How a class's columns are cut into work items (host planning, dry run):
every group's runs tile its columns, none is larger than the configured
columns, runs shrink only towards the end of a class, and small steps are cut
fine enough to give every CU something."""
import numpy as np
import pytest

import workdump
from paper_1603_06958_amd import inputs


@pytest.mark.parametrize("k,lo,hi,opt", [
    (2, 0, 9, {}), (5, 30, 40, {}), (65, 1, 900, {}), (300, 200, 300, {}), (700, 0, 1400, {}),
    (700, 0, 1400, dict(cols_per_item=1)), (900, 20, 60, dict(cols_per_item=7, tile_rows=64, step_values=40_000)),
    (1500, 250, 260, dict(tile_rows=128, step_values=200_000))])
def test_runs_tile_the_columns(k, lo, hi, opt):
    d, info = workdump.dry_run(inputs.random_family(k, lo, hi, seed=k), **opt)
    if k <= 700:
        workdump.check_coverage(d)
    cap = info.cols_per_item
    assert cap == opt.get("cols_per_item", cap)
    for r in d["ranges"]:
        for cls in range(4):
            items = d["items"][r["begin"][cls]:r["end"][cls]]
            by_group = {}
            for it in items:
                assert it["c0"] < it["c1"] <= it["c0"] + cap
                by_group.setdefault(int(it["group"]), []).append((int(it["c0"]), int(it["c1"])))
            cols = 0
            for g, runs in by_group.items():
                runs.sort()
                assert all(a[1] == b[0] for a, b in zip(runs, runs[1:]))
                # a run is cut short only where its group ends
                assert all(c1 - c0 >= min(cap, 4) for c0, c1 in runs[:-1])
                cols += runs[-1][1] - runs[0][0]
            if cols >= 1024 and cap >= 16:  # four columns for each of 256 CUs
                assert len(items) >= 200
            if len(items):  # whole runs at most: no more items than columns a run, plus one end a group
                assert len(items) <= cols // min(cap, 4) + len(by_group)


def test_large_classes_use_full_runs():
    # k = 6000: 94 groups of about 3,000 columns, far more than 128 columns a CU
    d, info = workdump.dry_run(inputs.random_family(6000, 40, 40, seed=3))
    n = np.array([int(i["c1"] - i["c0"]) for i in d["items"]])
    assert n.max() == info.cols_per_item == 128
    assert n[n == 128].sum() > 0.5 * n.sum()
