"""The staging launch of a batch of any size: the launch's shape and the spans
it covers on the CPU (the library's own arithmetic), and on the GPU sequences
whose column streams end at a span's edges and more sequences than a launch
has workgroups."""
import numpy as np
import pytest

import hostcode
import oracle
from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "staging.h"
using namespace famsa;
int main() {
  for (unsigned long long n : {1ull, 1000ull, (1ull << 22) - 1, 1ull << 22, (1ull << 22) + 1, (1ull << 24) - 1, 1ull << 24,
                               (1ull << 24) + 1, 20000000ull, 0xFFFFFFEFull, 0xFFFFFFEFull * 17}) {
    const unsigned long long b = stage_blocks(n);
    if (b == 0 || b > n || b * kStageThreads >= 1ull << 32) printf("%llu spans: %llu workgroups\n", n, b);
  }
  for (unsigned len = 0; len <= 65535; ++len) {  // the spans hold the stream, and none is empty
    const unsigned long long codes = stream_codes(len), spans = 1 + stage_more_spans(len);
    if (codes % 8 || codes < len + 8 || codes > len + 15 || spans * kStageSpan < codes || (spans - 1) * kStageSpan >= codes)
      printf("length %u: %llu codes in %llu spans\n", len, codes, spans);
  }
}
"""


def test_launch_shape(tmp_path):
    assert hostcode.run(tmp_path, PROGRAM) == ""


@pytest.mark.gpu
def test_streams_that_end_at_a_span():
    rng = np.random.default_rng(2)
    lens = [4079, 4080, 4081, 4087, 4088, 4089, 4095, 4096, 4097, 0, 1, 8176, 8184, 8185, 8192, 12281, 63, 64, 65]
    b = inputs.from_sequences([rng.integers(0, 20, n).astype(np.uint8) for n in lens])
    with B.Plan.from_batch(b) as p:
        tiles = p.collect()
    assert np.array_equal(tiles[(0, 0, len(lens))], oracle.tile_expected(b.codes, b.seq_off, 0, len(lens), 0, len(lens)))


@pytest.mark.gpu
def test_more_sequences_than_a_launch_holds():
    rng = np.random.default_rng(3)
    fam = [rng.integers(0, 20, n).astype(np.uint8) for n in (70, 4100, 300)]
    n1 = 1 << 24  # families of one sequence of one residue, between two of three sequences
    lens = np.concatenate([[s.size for s in fam], np.ones(n1, np.int64), [s.size for s in fam]])
    off = np.zeros(lens.size + 1, np.uint64)
    np.cumsum(lens, out=off[1:])
    codes = np.concatenate(fam + [np.zeros(n1, np.uint8)] + fam)
    fam_off = np.concatenate([[0], np.arange(3, n1 + 4), [n1 + 6]]).astype(np.uint32)
    want = oracle.tile_expected(codes[:int(off[3])], off[:4], 0, 3, 0, 3)
    got = []
    with B.Plan(codes, off, fam_off) as p:
        with pytest.raises(B.FamsaError):  # the first family's tile, then cancelled
            p.run(lambda t: got.append(B.tile_array(t).copy()) or 1)
        p.run(lambda t: got.append(B.tile_array(t).copy()), first_tile=n1 + 1)  # the last family's
    assert len(got) == 2 and np.array_equal(got[0], want) and np.array_equal(got[1], want)


SPACING = r"""
#include <cstdio>
#include "staging.h"
using namespace famsa;
int main() {
  for (unsigned len = 0; len <= 65535; ++len) {
    const unsigned long long apart = code_bytes(len, true), packed = code_bytes(len, false);
    if (packed != len || apart % 32 || apart < len || apart >= len + 32ull) printf("length %u: %llu, %llu\n", len, apart, packed);
  }
}
"""


def test_a_plain_plans_codes_lie_at_32_bytes(tmp_path):
    assert hostcode.run(tmp_path, SPACING) == ""


@pytest.mark.gpu
def test_codes_that_begin_past_the_callers_first():
    rng = np.random.default_rng(5)
    lens = [0, 1, 31, 32, 33, 64, 0, 95, 96, 97, 261]
    b = inputs.from_sequences([rng.integers(0, 20, n).astype(np.uint8) for n in lens])
    codes, off = np.concatenate([np.full(77, 19, np.uint8), b.codes]), b.seq_off + np.uint64(77)
    want = oracle.tile_expected(b.codes, b.seq_off, 0, len(lens), 0, len(lens))
    for flags in (0, B.PLAIN):
        with B.Plan(codes, off, flags=flags) as p:
            assert np.array_equal(p.collect()[(0, 0, len(lens))], want)
