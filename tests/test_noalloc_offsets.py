"""The allocation-free call reads no residue of a family with any invalid
length or offset: the verdict every staging workgroup takes before its first
read (the kernel's own function, its threads' shares joined by an AND), on the
CPU, and the call itself on families whose offsets go wrong in one place."""
import numpy as np
import pytest

import hostcode
from paper_1603_06958_amd import binding as B
from paper_1603_06958_amd import inputs

PROGRAM = r"""
#include <cstdio>
#include <vector>
#include "noalloc_input.h"
int main(int, char** a) {  // a file of k, maxlen and offsets, family after family; one verdict a family
  unsigned k, maxlen;
  if (!freopen(a[1], "r", stdin)) return 1;
  while (scanf("%u %u", &k, &maxlen) == 2) {
    std::vector<uint64_t> off(k + 1);
    for (auto& o : off) { unsigned long long x; if (scanf("%llu", &x) != 1) return 1; o = x; }
    bool ok = true;
    for (unsigned t = 0; t < 1024; ++t) ok = famsa::na_share_valid(off.data(), k, maxlen, t, 1024) && ok;
    printf("%d\n", ok);
  }
  static_assert(famsa::na_share_valid(nullptr, 0, 0, 0, 1024), "an empty family is valid");
}
"""


def families():
    rng = np.random.default_rng(1)
    out = [([0, 10, 2 ** 40, 2 ** 40 + 50], 896, False), ([0, 10, 20, 70], 896, True), ([0, 10, 5, 9], 896, False),
           ([2 ** 40, 2 ** 40 + 896], 896, True), ([0, 897], 896, False), ([0, 512], 512, True), ([0, 513], 512, False),
           ([2 ** 63, 2 ** 63 + 1, 0, 5], 896, False), ([5, 5, 5], 896, True), ([7], 896, True)]
    for k in (1023, 1024, 1025, 2048, 8192):  # a thread's last share, and its second one
        lens = rng.integers(0, 300, k)
        good = np.concatenate([[0], np.cumsum(lens)]).astype(np.uint64)
        out.append((good.tolist(), 512, True))
        for at in (0, 1, k // 2, k - 1, k):
            bad = good.copy()
            bad[at:] += np.uint64(600)
            out.append((bad.tolist(), 512, at == 0))
            if 0 < at < k:
                bad = good.copy()
                bad[at] = good[-1] + np.uint64(1)
                out.append((bad.tolist(), 512, False))
    return out


def test_one_invalid_offset_rejects_the_family(tmp_path):
    fams = families()
    (tmp_path / "in").write_text("\n".join(" ".join(map(str, [len(o) - 1, m] + o)) for o, m, _ in fams))
    got = hostcode.run(tmp_path, PROGRAM, tmp_path / "in").split()
    assert [g == "1" for g in got] == [ok for _, _, ok in fams]


@pytest.mark.gpu
@pytest.mark.parametrize("k", [3, 70, 1500, 4100])
def test_a_length_over_the_limit_between_valid_calls(k):
    import torch
    b = inputs.random_family(k, 20, 60, seed=k)
    total = int(b.seq_off[-1])
    codes = torch.full((total + 4096,), 200, dtype=torch.uint8, device="cuda")  # past the family: no code at all
    codes[:total] = torch.from_numpy(b.codes).cuda()
    n = k * (k - 1) // 2

    def call(off):
        out = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        status = torch.full((1,), -7, dtype=torch.int32, device="cuda")
        o = torch.from_numpy(off.astype(np.int64)).cuda()
        B.family_noalloc(codes.data_ptr(), o.data_ptr(), k, out.data_ptr(), status.data_ptr())
        torch.cuda.synchronize()
        return out.cpu().numpy(), int(status.item())

    want, st = call(b.seq_off)
    assert st == B.OK and (want >= 0).all()
    long, back = b.seq_off.copy(), b.seq_off.copy()
    long[k // 2 + 1:] += np.uint64(1000)  # what follows lies past the family, inside the buffer
    back[k // 2] = b.seq_off[-1]
    for off in (long, back, long):
        got, st = call(off)
        assert st == B.EINVAL and (got == -1).all()
        got, st = call(b.seq_off)
        assert st == B.OK and np.array_equal(got, want)
