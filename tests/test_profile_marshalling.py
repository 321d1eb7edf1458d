"""Arguments of profile_align as the library receives them, whatever arrays the
caller has: other types and orders, lists, empty problems."""
import numpy as np
import pytest

from paper_1603_06958_amd import binding as B


class Fake:
    """Stands in for the library call: keeps copies of the arrays behind the pointers."""

    def famsa_profile_align(self, n, seqs, seq_off, rows, rows_off, nrows, width, sigma, S, costs, device, score, ops,
                            ops_off, nops):
        so = np.ctypeslib.as_array(seq_off, (n + 1,)).copy()
        ro = np.ctypeslib.as_array(rows_off, (n + 1,)).copy()
        K, w = np.ctypeslib.as_array(nrows, (max(n, 1),)).copy(), np.ctypeslib.as_array(width, (max(n, 1),)).copy()
        s = np.ctypeslib.as_array(seqs, (max(int(so[-1]), 1),)).copy()
        r = np.ctypeslib.as_array(rows, (max(int(ro[-1]), 1),)).copy()
        oo = np.ctypeslib.as_array(ops_off, (n + 1,)).copy()
        out, cnt = np.ctypeslib.as_array(ops, (max(int(oo[-1]), 1),)), np.ctypeslib.as_array(nops, (max(n, 1),))
        self.got = [(s[so[p]:so[p + 1]], r[ro[p]:ro[p + 1]].reshape(K[p], w[p])) for p in range(n)]
        for p in range(n):
            assert oo[p + 1] - oo[p] == so[p + 1] - so[p] + w[p]
            cnt[p] = p % (int(oo[p + 1] - oo[p]) + 1)
            out[int(oo[p]):int(oo[p]) + int(cnt[p])] = p % 3
        return 0


@pytest.mark.parametrize("form", ["plain", "int64", "fortran", "strided", "mixed", "lists", "sliced"])
def test_every_form_of_input(form, monkeypatch):
    rng = np.random.default_rng(3)
    probs = [(rng.integers(0, 20, m).astype(np.uint8), rng.integers(0, 20, (K, n)).astype(np.uint8))
             for m, n, K in [(5, 7, 3), (0, 4, 1), (6, 0, 2), (1, 1, 1), (40, 33, 9)]]
    given = probs
    if form == "int64":
        given = [(a.astype(np.int64), r.astype(np.int64)) for a, r in probs]
    elif form == "fortran":
        given = [(a, np.asfortranarray(r)) for a, r in probs]
    elif form == "strided":
        given = [(np.repeat(a, 2)[::2], np.repeat(np.repeat(r, 2, 0), 3, 1)[::2, ::3]) for a, r in probs]
    elif form == "mixed":
        given = [(a.astype(np.int32), r) if i % 2 else (a, r.astype(np.uint16)) for i, (a, r) in enumerate(probs)]
    elif form == "lists":
        given = [(a.tolist(), r) for a, r in probs]
    elif form == "sliced":
        given = [(np.concatenate([a, a])[:a.size], np.concatenate([r, r])[:r.shape[0]]) for a, r in probs]
    fake = Fake()
    monkeypatch.setattr(B, "_lib", fake)
    for _ in range(2):  # the second call has the thread's scratch array already
        score, ops = B.profile_align(given, np.eye(20, dtype=np.int32), (1, 1, 1, 1))
        assert len(score) == len(ops) == len(probs)
        for (a, r), (ga, gr) in zip(probs, fake.got):
            assert np.array_equal(a, ga) and np.array_equal(r, gr)
        for p, o in enumerate(ops):
            assert o.dtype == np.uint8 and (o == p % 3).all() and o.base is None


def test_no_problems(monkeypatch):
    monkeypatch.setattr(B, "_lib", Fake())
    score, ops = B.profile_align([], np.eye(4, dtype=np.int32), (1, 1, 1, 1))
    assert len(score) == 0 and ops == []
