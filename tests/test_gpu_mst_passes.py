"""The GPU single-linkage consumer past one workgroup's components, on made-up
tiles whose values force what sequences rarely do: every pair of a tile
surviving the pass over it (so that it is split), ties everywhere, hook chains
as long as the family, more Boruvka rounds than the hierarchy keeps, tiles in
any order.  The forest must be the host Kruskal's, edge for edge."""
import ctypes

import numpy as np
import pytest
import torch  # before the library is loaded: both then use torch's HIP runtime

from paper_1603_06958_amd import binding as B

pytestmark = pytest.mark.gpu


def values(kind, k, rng):
    """Lengths and LCS(i, j) of every pair i < j (a k x k array)."""
    i, j = np.arange(k)[:, None], np.arange(k)[None, :]
    if kind == "random":
        lens = rng.integers(40, 300, k)
        return lens, rng.integers(0, 41, (k, k)).astype(np.int32)
    lens = np.full(k, 60000)
    if kind == "flat":
        return lens, np.full((k, k), 777, np.int32)
    if kind == "rising":  # a later row beats every earlier one
        return lens, np.broadcast_to(i + 1, (k, k)).astype(np.int32)
    if kind == "chain":  # the best partner is always the next sequence
        return lens, (30000 - 3 * abs(i - j) + np.minimum(i, j)).astype(np.int32)
    # halves: blocks of 2, 4, 8, ... ever less similar, a round for each
    x = np.bitwise_xor(i, j)
    return lens, (40000 - 1500 * np.floor(np.log2(np.maximum(x, 1))) - (i % 7)).astype(np.int32)


@pytest.mark.parametrize("kind,k,R,order", [
    ("random", 4096, 1024, "up"), ("random", 4097, 1500, "down"), ("random", 4300, 700, "mixed"),
    ("flat", 4200, 1024, "up"), ("rising", 4200, 4200, "up"), ("rising", 4200, 1024, "up"), ("chain", 4200, 1024, "up"),
    ("chain", 4200, 900, "down"), ("halves", 4096, 512, "mixed"), ("random", 129, 128, "up"), ("rising", 700, 300, "up")])
def test_forest_of_made_up_tiles(kind, k, R, order):
    rng = np.random.default_rng(k + R)
    lens, M = values(kind, k, rng)
    iu = np.triu_indices(k, 1)
    L = M[iu].astype(np.int64)
    d = lens[iu[0]] + lens[iu[1]] - 2 * L
    want = B.spanning_forest(k, iu[0], iu[1], L, d * d)
    starts = list(range(0, k, R))
    if order == "down":
        starts.reverse()
    elif order == "mixed":
        rng.shuffle(starts)
    m = B.Mst(lens.astype(np.uint32))
    stream = torch.cuda.Stream()
    for r0 in starts:
        r1 = min(k, r0 + R)
        host = np.concatenate([M[r, r + 1:] for r in range(r0, r1)])
        tile = torch.from_numpy(host).cuda()
        torch.cuda.synchronize()
        t = B.Tile(tile_index=r0 // R, family=0, k=k, row_begin=r0, row_end=r1, count=host.size,
                   lcs=ctypes.cast(tile.data_ptr(), ctypes.POINTER(ctypes.c_int32)), stream=stream.cuda_stream, values=0)
        assert B.lib().famsa_mst_consume(m.handle, ctypes.byref(t)) == 0, B.last_error()
        tile.fill_(-1)  # the call has finished reading the tile
    got = m.result()
    m.close()
    assert sorted(zip(*[x.tolist() for x in got])) == sorted(zip(*[x.tolist() for x in want]))
