"""Device blocks kept between objects: results do not depend on what a block
held before, objects on several threads never share one, and the store gives
its blocks back (it is bounded, and emptied before an allocation fails)."""
import threading

import numpy as np
import pytest
import torch  # before the library is loaded: both then use torch's HIP runtime

import oracle
from oracle import gapped as G
from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

pytestmark = pytest.mark.gpu


def decode_all(seqs, cols, lens):
    off = np.zeros(len(seqs) + 1, np.uint64)
    np.cumsum([s.size for s in seqs], out=off[1:])
    gp = B.Gapped(np.concatenate(seqs), off)
    gp.insert(cols, lens)
    w, rows = gp.width(), gp.decode()
    gp.close()
    return w, rows


def test_rows_past_the_width_are_zero_whatever_the_block_held():
    rng = np.random.default_rng(1)
    for rnd in range(4):  # large enough for kept blocks: over 1 MB of rows
        seqs = [rng.integers(1, 20, int(n)).astype(np.uint8) for n in rng.integers(5, 700, 3000)]
        cols, lens = [1, 4], [int(x) for x in rng.integers(1, 5, 2)]
        w, rows = decode_all(seqs, cols, lens)
        for i in range(0, 3000, 211):
            s = G.insert_runs(G.from_symbols(seqs[i].tolist()), list(zip(cols, lens)))
            want = [0xFF if c is None else c for c in s[1:]]
            assert rows[i, :w[i]].tolist() == want
            assert not rows[i, w[i]:].any()


def test_threads_with_their_own_objects():
    b = inputs.random_family(700, 30, 90, seed=5)
    want = oracle.tile_expected(b.codes, b.seq_off, 0, 700, 0, 700)
    fams = [inputs.c2(k=2500, root_len=40, seed=s) for s in (1, 2)]
    bad = []

    def tree(f):
        m = B.Mst(f.lengths())
        with B.Plan.from_batch(f, flags=B.DEVICE_TILES) as p:
            p.run_native(B.Mst.consume_fn(), m.handle)
        t = m.guide_tree()
        m.close()
        return [x.tolist() for x in t]

    ref = [tree(f) for f in fams]

    def work(i):
        for _ in range(4):
            if i < 2:
                if tree(fams[i]) != ref[i]:
                    bad.append(i)
            else:
                with B.Plan.from_batch(b) as p:
                    got = p.collect()
                if not np.array_equal(got[(0, 0, 700)], want):
                    bad.append(i)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def test_store_is_bounded_and_given_back():
    lens = np.full(200_000, 10, np.uint32)  # a block of about 200 MB each
    B.Mst(lens).close()
    free0 = torch.cuda.mem_get_info(0)[0]
    for _ in range(3):
        ms = [B.Mst(lens) for _ in range(4)]
        for m in ms:
            m.close()
    assert free0 - torch.cuda.mem_get_info(0)[0] <= 512 << 20
    # a budget counts the kept blocks as free, and an allocation that needs them gets them
    b = inputs.random_family(50, 10, 20, seed=1)
    with B.Plan.from_batch(b) as p:
        assert p.collect()
