"""Plans made and run, forests read and gapped sequences decoded by several
threads at once, each with objects of its own (blocks of over a megabyte among
them, which are kept when they are released): no call fails, none spoils
another thread's graphs, and every result is the one a single thread gets."""
import threading

import numpy as np
import pytest
import torch  # before the library is loaded: both then use torch's HIP runtime

from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

pytestmark = pytest.mark.gpu


def tiles(b):
    with B.Plan.from_batch(b) as p:
        return [x.tolist() for x in p.collect().values()]


def tree(b):
    m = B.Mst(b.lengths())
    with B.Plan.from_batch(b, flags=B.DEVICE_TILES, tile_rows=300) as p:
        p.run_native(B.Mst.consume_fn(), m.handle)
    t = [x.tolist() for x in m.guide_tree()] + [list(m.stats())[:1]]
    m.close()
    return t


def gapped(b):
    g = B.Gapped(b.codes, b.seq_off)
    g.insert([1, 3], [2, 1])
    out = [x.tolist() for x in g.state(b.nseq - 1)] + [g.decode().tolist()]
    g.close()
    return out


def test_threads_with_objects_of_their_own():
    small, long = inputs.random_family(60, 10, 300, seed=1), inputs.random_family(900, 20, 60, seed=2)
    work = [(tiles, small), (tree, small), (tree, long), (gapped, long), (tiles, long), (tree, small)]
    want = [f(b) for f, b in work]
    errors = []

    def run(i):
        f, b = work[i]
        try:
            for n in range(12):
                if f(b) != want[i]:
                    errors.append(f"{f.__name__} {i}, pass {n}: another result")
        except Exception as e:  # a thread's own exceptions are not the test's
            errors.append(f"{f.__name__} {i}: {e}")

    ts = [threading.Thread(target=run, args=(i,)) for i in range(len(work))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not errors, errors
