"""Tiles in descending order, a family in one tile and tiles that overlap what
the forest joins: the consumer takes their rows from the last one up, blocks of
them tied to the forest before their pass.  Block sizes either side of the
first one's, values that let every pair through (a block that does not fit) or
hardly any; the forest must be the host Kruskal's, edge for edge, and tiles in
descending order must not cost an update each."""
import ctypes

import numpy as np
import pytest
import torch  # before the library is loaded: both then use torch's HIP runtime

from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

pytestmark = pytest.mark.gpu


def values(kind, k, rng):
    """Lengths and LCS(i, j) of every pair i < j (a k x k array)."""
    i, j = np.arange(k)[:, None], np.arange(k)[None, :]
    if kind == "random":
        return rng.integers(40, 300, k), rng.integers(0, 41, (k, k)).astype(np.int32)
    lens = np.full(k, 60000)
    if kind == "same":  # identical sequences: every similarity infinite
        return lens, np.full((k, k), 60000, np.int32)
    if kind == "none":  # nothing in common with anything
        return lens, np.zeros((k, k), np.int32)
    if kind == "flat":
        return lens, np.full((k, k), 777, np.int32)
    if kind == "falling":  # an earlier row beats every later one
        return lens, np.broadcast_to(k - i, (k, k)).astype(np.int32)
    # blocks of 2, 4, 8, ... ever less similar, a round for each
    x = np.bitwise_xor(i, j)
    return lens, (40000 - 1500 * np.floor(np.log2(np.maximum(x, 1))) - (i % 7)).astype(np.int32)


def forest(lens, M, tiles):
    k = len(lens)
    m = B.Mst(lens.astype(np.uint32))
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for n, (r0, r1) in enumerate(tiles):
        host = np.concatenate([M[r, r + 1:] for r in range(r0, r1)])
        tile = torch.from_numpy(host).cuda()
        torch.cuda.synchronize()
        t = B.Tile(tile_index=n, family=0, k=k, row_begin=r0, row_end=r1, count=host.size,
                   lcs=ctypes.cast(tile.data_ptr(), ctypes.POINTER(ctypes.c_int32)), stream=streams[n & 1].cuda_stream,
                   values=0)
        assert B.lib().famsa_mst_consume(m.handle, ctypes.byref(t)) == 0, B.last_error()
        tile.fill_(-1)  # the call has finished reading the tile
    got = m.result()
    m.close()
    return sorted(zip(*[x.tolist() for x in got]))


def kruskal(lens, M, lo):
    k = len(lens)
    iu = np.triu_indices(k, 1)
    on = iu[0] >= lo
    i, j = iu[0][on], iu[1][on]
    L = M[i, j].astype(np.int64)
    d = lens[i] + lens[j] - 2 * L
    return sorted(zip(*[x.tolist() for x in B.spanning_forest(k, i, j, L, d * d)]))


def down(k, R, lo=0):
    return [(r0, min(k, r0 + R)) for r0 in range(lo, k, R)][::-1]


@pytest.mark.parametrize("kind", ["random", "same", "none", "flat", "falling", "halves"])
@pytest.mark.parametrize("k,tiles", [
    (3, down(3, 1)), (130, down(130, 1)), (128, [(0, 128)]), (129, [(0, 129)]), (130, [(0, 130)]), (1024, [(0, 1024)]),
    (1100, [(0, 1100)]), (700, down(700, 97)), (1500, down(1500, 257)), (1500, down(1500, 1024, 5)),
    (4300, [(0, 4300)]), (4300, down(4300, 1024)),
    (900, [(500, 900), (300, 700), (300, 700), (0, 310)]),        # rows that were there, again
    (900, [(600, 900), (0, 200), (200, 600)]), (900, [(899, 900), (0, 899)])])
def test_rows_from_the_last_one_up(kind, k, tiles):
    lens, M = values(kind, k, np.random.default_rng(k))
    assert forest(lens, M, tiles) == kruskal(lens, M, min(r0 for r0, _ in tiles))


def test_descending_tiles_share_updates():
    b = inputs.random_family(3000, 60, 60, seed=4)
    rounds = {}
    for flags in (0, B.DESCENDING):
        m = B.Mst(b.lengths())
        with B.Plan.from_batch(b, flags=B.DEVICE_TILES | flags, tile_rows=250) as p:
            p.run_native(B.Mst.consume_fn(), m.handle)
        rounds[flags] = m.stats()[1]
        m.close()
    # an update is at most a dozen rounds; five of them are the first rows', the first tile's and the waiting survivors'
    assert rounds[B.DESCENDING] <= 60, rounds


@pytest.mark.parametrize("k,tiles", [(2600, [(0, 2600)]), (2600, down(2600, 512)), (1200, [(0, 1200)])])
def test_clades_one_after_another(k, tiles):
    """A family listed clade by clade: rows unlike all that the forest holds, and like each other."""
    rng = np.random.default_rng(k)
    clade = np.sort(rng.integers(0, 7, k))
    M = np.where(clade[:, None] == clade[None, :], 30000, 500).astype(np.int32) + rng.integers(0, 400, (k, k)).astype(np.int32)
    lens = np.full(k, 60000)
    assert forest(lens, M, tiles) == kruskal(lens, M, 0)
