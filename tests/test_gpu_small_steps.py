"""Steps whose length classes share one launch, and the allocation-free call
either side of it: the smallest families, the item counts at which the launch
changes, groups with a single row, widths at the ends of every class; values
are the oracle's (or the plain kernel's where there are many)."""
import numpy as np
import pytest
import torch  # before the library is loaded: both then use torch's HIP runtime

import oracle
from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

pytestmark = pytest.mark.gpu


def triangle(tiles, k):
    return np.concatenate([tiles[key] for key in sorted(tiles)]) if tiles else np.zeros(0, np.int32)


def noalloc(b, sigma):
    k = b.nseq
    codes = torch.from_numpy(np.append(b.codes, np.uint8(0))).cuda()
    off = torch.from_numpy(b.seq_off.astype(np.int64)).cuda()
    out = torch.full((max(1, k * (k - 1) // 2),), -7, dtype=torch.int32, device="cuda")
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    B.family_noalloc(codes.data_ptr(), off.data_ptr(), k, out.data_ptr(), status.data_ptr(), alphabet_size=sigma)
    torch.cuda.synchronize()
    return out.cpu().numpy()[:k * (k - 1) // 2], int(status.item())


@pytest.mark.parametrize("k,sigma", [(2, 20), (3, 32), (63, 20), (64, 20), (65, 20), (66, 32), (129, 20), (200, 32)])
def test_mixed_classes_match_the_oracle(k, sigma):
    rng = np.random.default_rng(k)
    edge = [0, 1, 31, 32, 33, 255, 256, 257, 383, 384, 385, 511, 512] + ([] if sigma > 20 else [640, 895, 896])
    lens = [edge[i % len(edge)] for i in range(k)]
    b = inputs.from_sequences([rng.integers(0, sigma, n).astype(np.uint8) for n in lens])
    want = oracle.tile_expected(b.codes, b.seq_off, 0, k, 0, k)
    for flags in (0, B.NO_GRAPH):
        with B.Plan.from_batch(b, alphabet_size=sigma, flags=flags) as p:
            assert np.array_equal(triangle(p.collect(), k), want)
    got, status = noalloc(b, sigma)
    assert status == 0 and np.array_equal(got, want)


# item counts around twice the CU count of 256: one launch below, a launch a class above
@pytest.mark.parametrize("k", [900, 1000, 1100, 1300, 2000])
def test_launch_change(k):
    b = inputs.random_family(k, 0, 420, seed=k)
    with B.Plan.from_batch(b, flags=B.PLAIN) as p:
        want = triangle(p.collect(), k)
    with B.Plan.from_batch(b) as p:
        assert np.array_equal(triangle(p.collect(), k), want)
    for _ in range(2):
        got, status = noalloc(b, 20)
        assert status == 0 and np.array_equal(got, want)


@pytest.mark.parametrize("k", [70, 1500])
def test_invalid_codes_between_valid_calls(k):
    b = inputs.random_family(k, 20, 90, seed=k)
    bad = inputs.Batch(b.codes.copy(), b.seq_off, b.fam_off)
    bad.codes[int(b.seq_off[k // 2])] = 200
    want, _ = noalloc(b, 20)
    for b2, ok in ((bad, False), (b, True), (bad, False), (bad, False), (b, True), (b, True)):
        got, status = noalloc(b2, 20)
        assert status == (0 if ok else B.EINVAL)
        assert np.array_equal(got, want) if ok else (got == -1).all()


def test_server_steps_of_one_launch():
    from paper_1603_06958_amd import serve
    jobs = [inputs.random_family(k, 0, 500, seed=k) for k in (2, 5, 40, 90)]
    srv, got = serve.Server(), {}
    ids = [srv.submit(b.codes, b.seq_off) for b in jobs]

    def take(t):
        got.setdefault(int(t.family), []).append(B.tile_array(t).copy())
        return 0

    while srv.step(take):
        pass
    srv.close()
    for i, b in zip(ids, jobs):
        assert np.array_equal(np.concatenate(got[i]), oracle.tile_expected(b.codes, b.seq_off, 0, b.nseq, 0, b.nseq))
