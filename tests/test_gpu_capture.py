"""Another thread's graph capture (thread-local mode, so that only its own
thread's calls concern it) goes on while every kind of object is made, used and
released beside it: no call waits for the whole device or uses the null stream,
which would fail and spoil the capture.  Blocks of over a megabyte, kept when
they are released, are among the objects' memory."""
import threading

import numpy as np
import pytest
import torch  # before the library is loaded: both then use torch's HIP runtime

from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs
from paper_1603_06958_amd.serve import Server

pytestmark = pytest.mark.gpu

FAMILY = inputs.random_family(900, 20, 60, seed=2)  # 1.6 MB of results, a forest of 1.9 MB


def tiles(flags=0):
    with B.Plan.from_batch(FAMILY, flags=flags, tile_rows=300) as p:
        p.collect()


def tuned():
    with B.Plan.from_batch(FAMILY, flags=B.NO_AUTOTUNE) as p:
        p.autotune()


def tree():
    m = B.Mst(FAMILY.lengths())
    with B.Plan.from_batch(FAMILY, flags=B.DEVICE_TILES, tile_rows=300) as p:
        p.run_native(B.Mst.consume_fn(), m.handle)
    m.guide_tree()
    m.result()
    m.stats()
    m.close()


def gapped():
    g = B.Gapped(FAMILY.codes, FAMILY.seq_off)
    g.insert([1, 3], [2, 1])
    g.locate(np.arange(4), np.arange(4))
    g.state(5)
    g.decode()
    g.close()


def profile():
    rng = np.random.default_rng(3)
    problems = [inputs.profile_problem(300, 300, 40, rng) for _ in range(20)]
    B.profile_align([(p.seq, p.rows) for p in problems], inputs.synthetic_subst(20, 1), (1, 1, 1, 1))


def serve():
    s = Server(tile_rows=256, step_values=1 << 20)
    s.submit(FAMILY.codes, FAMILY.seq_off)
    while s.step():
        pass
    s.close()


def peak():
    B.valu_peak(iters=64)


WORK = [tiles, lambda: tiles(B.TWO_STREAMS), lambda: tiles(B.PLAIN), tuned, tree, gapped, profile, serve, peak, B.trim]


@pytest.mark.parametrize("i", range(len(WORK)))
def test_another_threads_capture_goes_on(i):
    x = torch.zeros(1000, device="cuda")
    graph, errors = torch.cuda.CUDAGraph(), []

    def work():
        try:
            WORK[i]()
        except Exception as e:
            errors.append(repr(e))

    torch.cuda.synchronize()
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        graph.capture_begin(capture_error_mode="thread_local")
        try:
            x += 1
            t = threading.Thread(target=work)
            t.start()
            t.join()
            x += 2
        finally:
            graph.capture_end()
    assert not errors, errors
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
    assert x.eq(9).all()
