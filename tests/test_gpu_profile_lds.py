"""The sequence-to-profile DP where its inputs just fit a CU's LDS and just do
not (int16 and int32 cost tables, int32 and int64 values), alone and with more
problems than CUs (half of the LDS each): scores and alignments are the
oracle's."""
import numpy as np
import pytest

from oracle import profile as OP
from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sigma,n,K,scale,extra", [
    # bytes a column: 16 (record) + 32 (edge rows) + 2 or 4 sigma (costs) in int32, twice the first two in int64;
    # the CU's 160 KB less the kernel's own: about 1,770 columns of 88, 1,220 of 128, 885 of 176
    (20, 1740, 3, 1, 0), (20, 1790, 3, 1, 0), (20, 1210, 40, 90, 0), (20, 1240, 40, 90, 0),
    (20, 870, 30, 100000, 0), (20, 900, 30, 100000, 0), (20, 860, 3, 1, 260), (20, 940, 3, 1, 260)])
def test_either_side_of_the_lds(sigma, n, K, scale, extra):
    rng = np.random.default_rng(n + K)
    S = inputs.synthetic_subst(sigma, 5) * (min(scale, 80))
    costs = tuple(c * scale for c in (9, 2, 8, 3))
    probs = [inputs.profile_problem(70, n, K, rng, alphabet=sigma), inputs.profile_problem(33, 40, 2, rng, alphabet=sigma)]
    probs += [inputs.profile_problem(9, 11, 2, rng, alphabet=sigma) for _ in range(extra)]
    got_s, got_ops = B.profile_align([(p.seq, p.rows) for p in probs], S, costs)
    for q, p in enumerate(probs):
        exp_s, exp_ops = OP.align(p.seq, p.rows, S, costs)
        assert int(got_s[q]) == exp_s
        assert got_ops[q].tolist() == exp_ops
