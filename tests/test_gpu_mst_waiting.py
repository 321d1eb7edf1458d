"""The GPU single-linkage consumer's list of survivors over several tiles:
thin tiles that wait together, a pair given more than once before it is taken
in, the forest read between tiles and by several threads, a pass that finds
the list full.  The forest must be the host Kruskal's of the tiles so far."""
import ctypes
import threading

import numpy as np
import pytest
import torch  # before the library is loaded: both then use torch's HIP runtime

from paper_1603_06958_amd import binding as B

pytestmark = pytest.mark.gpu


def consume(m, M, r0, r1, stream):
    k = M.shape[0]
    host = np.concatenate([M[r, r + 1:] for r in range(r0, r1)])
    tile = torch.from_numpy(host).cuda()
    torch.cuda.synchronize()
    t = B.Tile(tile_index=0, family=0, k=k, row_begin=r0, row_end=r1, count=host.size,
               lcs=ctypes.cast(tile.data_ptr(), ctypes.POINTER(ctypes.c_int32)), stream=stream.cuda_stream, values=0)
    assert B.lib().famsa_mst_consume(m.handle, ctypes.byref(t)) == 0, B.last_error()
    tile.fill_(-1)  # the call has finished reading the tile


def edges(e):
    return sorted(zip(*[x.tolist() for x in e]))


def kruskal(lens, M, upto):
    k = len(lens)
    iu = np.triu_indices(k, 1)
    on = iu[0] < upto
    i, j = iu[0][on], iu[1][on]
    L = M[i, j].astype(np.int64)
    d = lens[i] + lens[j] - 2 * L
    return edges(B.spanning_forest(k, i, j, L, d * d))


@pytest.mark.parametrize("k,first,R,times", [
    (700, 64, 16, 2),     # one workgroup's components
    (4300, 128, 97, 2),   # rounds on the whole GPU; every tile twice
    (4300, 128, 400, 1),
    (2, 1, 1, 3), (65, 8, 1, 3)])
def test_tiles_that_wait(k, first, R, times):
    rng = np.random.default_rng(k + R)
    lens = rng.integers(40, 300, k)
    M = rng.integers(0, 41, (k, k)).astype(np.int32)
    m = B.Mst(lens.astype(np.uint32))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    starts = [0] + list(range(first, k, R))
    for n, r0 in enumerate(starts):
        r1 = min(k, first if r0 == 0 else r0 + R)
        for x in range(times):
            consume(m, M, r0, r1, streams[(n + x) & 1])
        if n in (1, len(starts) // 2):
            assert edges(m.result()) == kruskal(lens, M, r1)
    got = [None] * 4
    ts = [threading.Thread(target=lambda x=x: got.__setitem__(x, edges(m.result()))) for x in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    want = kruskal(lens, M, k)
    assert all(g == want for g in got)
    m.close()


def test_list_full_while_tiles_wait():
    """Rows that beat every row before: each tile's pairs all survive, more of
    them than there is room for behind the survivors that wait."""
    k = 4200
    lens = np.full(k, 60000)
    M = np.broadcast_to(np.arange(k)[:, None] + 1, (k, k)).astype(np.int32)
    m = B.Mst(lens.astype(np.uint32))
    s = torch.cuda.Stream()
    consume(m, M, 0, 300, s)
    r0 = 300
    for n in (1, 25, 1, 29, 120):  # room for about 30 rows
        consume(m, M, r0, r0 + n, s)
        r0 += n
    assert edges(m.result()) == kruskal(lens, M, r0)
    m.close()
