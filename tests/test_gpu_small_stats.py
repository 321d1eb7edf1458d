"""Launches and times of a step whose length classes share one launch."""
import pytest

from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lens,want", [((200, 300, 500, 1000), [0, 0, 1, 1]), ((200, 300), [0, 1, 0, 0]),
                                       ((200,), [1, 0, 0, 0])])
def test_one_launch_counts_once(lens, want):
    import numpy as np
    rng = np.random.default_rng(1)
    b = inputs.from_sequences([rng.integers(0, 20, n).astype(np.uint8) for n in lens for _ in range(70)])
    with B.Plan.from_batch(b, flags=B.NO_GRAPH | B.DEVICE_TILES) as p:
        for _ in range(2):
            p.run(lambda t: 0)
            s = p.stats()
            assert s.steps == 1 and list(s.launches)[:4] == want
            assert all((ms > 0) == (n > 0) for ms, n in zip(s.kernel_ms, s.launches))
            assert [c > 0 for c in s.cells][:4] == [any(lo < n <= hi for n in lens) for lo, hi in
                                                    ((0, 256), (256, 384), (384, 896), (896, 9999))]
