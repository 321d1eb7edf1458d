"""Gap insertion with as many runs as one group of lanes takes, one more and
one fewer (4, 16 and 64 lanes a sequence, several groups' worth), repeated
columns and empty runs among them, into sequences whose trees have different
depths: counters, trees and rows are the oracle's."""
import numpy as np
import pytest

from oracle import gapped as G
from paper_1603_06958_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nruns", [1, 3, 4, 5, 15, 16, 17, 63, 64, 65, 129, 200])
def test_runs_per_group(nruns):
    rng = np.random.default_rng(nruns)
    lens = [70, 0, 1, 300, 31, 32, 33, 1000, 255, 256, 5] + [int(x) for x in rng.integers(0, 200, 60)]
    seqs = [rng.integers(0, 20, n).astype(np.uint8) for n in lens]
    off = np.zeros(len(seqs) + 1, np.uint64)
    np.cumsum([s.size for s in seqs], out=off[1:])
    gp = B.Gapped(np.concatenate(seqs), off)
    strings = [G.from_symbols(s.tolist()) for s in seqs]
    for first, count in ((0, len(seqs)), (3, 1), (3, 40)):
        width = min(len(strings[i]) for i in range(first, first + count))
        cols = sorted(int(x) for x in rng.integers(1, width + 1, nruns))
        runs = [int(x) for x in rng.integers(0, 4, nruns)]
        gp.insert(cols, runs, first, count)
        for i in range(first, first + count):
            strings[i] = G.insert_runs(strings[i], list(zip(cols, runs)))
    assert list(gp.width()) == [len(s) - 1 for s in strings]
    for i, s in enumerate(strings):
        gaps, dps = gp.state(i)
        eg, ed = G.no_gaps(s), G.dps(s)
        assert gaps.tolist() == list(eg), i
        assert dps[1:].tolist() == list(ed)[1:], i
    gp.close()
