"""Work items are cut for as many workgroups as share a class: four a CU for
rows of up to 128 residues, three up to 256, two up to 384, one beyond (for 20
symbols), and for
fewer where the rows are so short or so few that an item would hold next to
nothing.  Host planning by dry runs, the allocation-free call's own functions
on the CPU, and values on the GPU at sizes either side of the rules."""
import numpy as np
import pytest

import hostcode
import workdump
from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

CUS = 256


@pytest.mark.parametrize("k,L,sigma,per_cu", [
    (2900, 100, 20, 4), (2000, 200, 20, 3), (3500, 250, 20, 3), (2000, 300, 20, 2), (2000, 380, 20, 2), (2000, 700, 20, 1),
    (2900, 150, 32, 2), (2000, 300, 32, 1)])
def test_no_item_is_more_than_a_slot(k, L, sigma, per_cu):
    d, _ = workdump.dry_run(inputs.random_family(k, L, L, seed=k, alphabet=sigma), alphabet_size=sigma)
    n = d["items"]["c1"].astype(int) - d["items"]["c0"]
    assert n.max() <= max(16, n.sum() / (CUS * per_cu))
    assert n.size >= CUS * per_cu  # every slot has something


@pytest.mark.parametrize("k,L", [(700, 30), (1000, 60), (5000, 30)])
def test_short_rows_in_fewer_items(k, L):
    d, _ = workdump.dry_run(inputs.random_family(k, L, L, seed=k))
    n = d["items"]["c1"].astype(int) - d["items"]["c0"]
    slots = max(CUS, min(4 * CUS, n.sum() * L / (500 * 8)))
    # guided runs: a slot's share of what is left each time, and the shortest ones at the end
    least = min(max(16, 1600 // L), max(4, n.sum() // int(slots)))
    assert n.size <= slots * (np.log(max(1.0, n.sum() / slots / least)) + 2) + n.sum() / 112 + k / 64
    assert np.median(n) >= least - 15  # whole multiples of 16 above that


PROGRAM = r"""
#include <cstdio>
#include <initializer_list>
#include "noalloc_input.h"
using namespace famsa;
int main() {
  for (uint32_t k = 0; k <= 8192; ++k) {
    const uint32_t most = na_all_items(k, na_runs_most());
    if (most > 8192) printf("%u sequences: %u items\n", k, most);  // the item array
    uint32_t cols = 0;
    for (uint32_t g = 0; g < na_groups(k); ++g) cols += k - (64 * g + 1);
    if (cols != na_columns(k, 0)) printf("%u sequences: %u columns\n", k, cols);
    for (uint64_t residues : {0ull, 1ull, 30ull * k, 100ull * k, 250ull * k, 896ull * k, ~0ull})
      for (uint32_t resident : {0u, 1u, 255u, 256u, 300u, 512u, 1024u, 0xFFFFFFFFu}) {
        const NaRuns r = na_runs(k, residues, resident);
        if (r.shift < 8 || r.shift > 10 || (r.shift > 8 && (3u << (r.shift - 2)) > resident)) printf("%u: shift %u\n", k, r.shift);
        uint32_t n = 0;
        for (uint32_t g = 0; g < na_groups(k); ++g) {
          const uint32_t c = na_cols(k, g, r), want = na_columns(k, g) >> r.shift;
          if (c == 0 || c > kNaColsMost || (c > 16 && c > want && c > r.floor && r.shift > 8)) printf("%u: runs of %u\n", k, c);
          n += na_items(k, g, c);
        }
        if (n > most) printf("%u sequences, %llu residues, %u: %u items, not %u\n", k, (unsigned long long)residues, resident, n, most);
      }
  }
  // 2,500 sequences of 250 residues: four a CU where the GPU holds that many; 50 of 30 do not need them
  if (na_runs(2500, 2500 * 250, 1024).shift != 10 || na_runs(2500, 2500 * 250, 512).shift != 9 ||
      na_runs(2500, 2500 * 250, 768).shift != 10 || na_runs(2500, 2500 * 250, 256).shift != 8 || na_runs(1200, 1200 * 30, 1024).shift != 8) printf("slots\n");
}
"""


def test_runs_of_the_allocation_free_call(tmp_path):
    assert hostcode.run(tmp_path, PROGRAM) == ""


@pytest.mark.gpu
@pytest.mark.parametrize("k,lo,hi,sigma", [(1100, 10, 40, 20), (1700, 200, 300, 20), (2600, 240, 260, 20),
                                           (1200, 370, 400, 20), (2100, 100, 300, 32), (8162, 5, 60, 20)])
def test_values_either_side(k, lo, hi, sigma):
    import torch
    b = inputs.random_family(k, lo, hi, seed=k, alphabet=sigma)
    n = k * (k - 1) // 2
    got = {}
    for flags in (B.PLAIN, 0):
        with B.Plan.from_batch(b, alphabet_size=sigma, flags=flags) as p:
            tiles = p.collect()
        got[flags] = np.concatenate([tiles[key] for key in sorted(tiles)])
    assert np.array_equal(got[0], got[B.PLAIN])
    codes = torch.from_numpy(b.codes).cuda()
    off = torch.from_numpy(b.seq_off.astype(np.int64)).cuda()
    out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    B.family_noalloc(codes.data_ptr(), off.data_ptr(), k, out.data_ptr(), status.data_ptr(), alphabet_size=sigma)
    torch.cuda.synchronize()
    assert int(status.item()) == 0 and np.array_equal(out.cpu().numpy(), got[B.PLAIN])


@pytest.mark.parametrize("k,lo,hi,sigma,flags", [
    (500, 1000, 1000, 20, B.LONG_SEGMENTED), (120, 900, 3000, 20, B.LONG_SEGMENTED), (300, 600, 900, 32, B.LONG_SEGMENTED),
    (40, 5000, 5000, 20, B.LONG_SEGMENTED), (700, 1000, 1000, 20, B.LONG_SEGMENTED), (300, 2000, 2000, 32, 0),
    (200, 6000, 6000, 20, 0), (100, 15000, 15000, 32, 0), (20, 15000, 15000, 32, 0), (500, 700, 700, 20, 0)])
def test_no_second_round_for_a_few_items(k, lo, hi, sigma, flags):
    """One workgroup a CU: a class whose columns fit in as many runs of sixteen has no more items than that, and the
    shortest such runs; one that is larger has none shorter than sixteen, but at the end of a group."""
    d, info = workdump.dry_run(inputs.random_family(k, lo, hi, seed=k, alphabet=sigma), alphabet_size=sigma, flags=flags)
    workdump.check_coverage(d)
    widest = 28 if sigma <= 20 else 16
    cols, runs = {}, {}
    for it in d["items"]:
        g = int(it["group"])
        if d["groups"][g]["W"] > widest or lo == 700:
            cols[g] = cols.get(g, 0) + int(it["c1"] - it["c0"])
            runs.setdefault(g, []).append(int(it["c1"] - it["c0"]))

    def items(n):
        return sum(-(-c // n) for c in cols.values())

    n_items = sum(len(r) for r in runs.values())
    if items(16) <= CUS:
        assert n_items <= CUS
        least = next(n for n in range(4, 17) if items(n) <= CUS)
        assert n_items == items(least)
    else:
        assert all(min(r[:-1], default=16) >= 16 for r in runs.values())
