// What the allocation-free call checks of its offsets before a residue is read,
// and how it cuts a family's columns into work items (constant expressions, so
// that the kernel and the host run the same code).
#pragma once
#include <stdint.h>

namespace famsa {

// One thread's share (sequences first, first + step, ...) of the check of a
// whole family: offsets that do not decrease, no sequence longer than maxlen.
// With every share valid all sequences lie between seq_off[0] and seq_off[k];
// with any other not, a sequence that is valid by itself may lie anywhere.
constexpr bool na_share_valid(const uint64_t* seq_off, uint32_t k, uint32_t maxlen, uint32_t first, uint32_t step) {
  bool ok = true;
  for (uint32_t i = first; i < k; i += step) {
    const uint64_t a = seq_off[i], b = seq_off[i + 1];
    ok &= !(b < a || b - a > maxlen);
  }
  return ok;
}

// Columns that the 64-row groups from `g` on walk: group h needs the positions
// after its own first row, [64 h + 1, k).
constexpr uint32_t na_groups(uint32_t k) { return k >= 2 ? (k - 2) / 64 + 1 : 0; }  // those with a pair: 64 h + 1 < k
constexpr uint32_t na_columns(uint32_t k, uint32_t g) {
  const uint32_t G = na_groups(k);
  return g >= G ? 0 : (G - g) * (k - 1) - 64 * ((G - 1) * G / 2 - (g * g - g) / 2);
}
// Work items, cut as the plan path cuts them (build_step): a group's columns in
// runs of 1 / slots of what is left, kNaColsMost at most (which keeps 8,192
// sequences within the item array).  slots: the workgroups that share a class,
// the power of two nearest to those the GPU holds at once (3, 2 and 1 a CU in
// the classes 0 to 2; 2, 1 and 1 over 20 symbols) while each gets kNaSlotWork
// residues of columns, one a CU at least.  floor: the shortest run worth its
// place in the queue, by the columns' mean length.
// 2,500 sequences of 250 residues (classes 0 and 1): 659 us cut for one
// workgroup a CU in every class, 570 in uniform runs of 16, 477 for four; but
// 1,200 of 700 (class 2, one a CU): 826, 840 and 1,001.
constexpr uint32_t kNaColsMost = 96;
constexpr float kNaSlotWork = 4000.0f, kNaLeastWork = 1600.0f;
struct NaRuns {
  uint32_t shift;  // slots = 2^shift: 256, 512 or 1024
  uint32_t floor;
};
// `resident`: workgroups of the group's class that the GPU holds.  Any value
// of `residues` (an invalid family's is not looked at before) gives one of the
// numbers of slots above.
constexpr NaRuns na_runs(uint32_t k, uint64_t residues, uint32_t resident) {
  const float len = (float)residues / (float)(k ? k : 1), slots = (float)na_columns(k, 0) * len / kNaSlotWork;
  NaRuns r{8, 0};
  while (r.shift < 10 && resident >= (3u << (r.shift - 1)) && slots >= 1.4f * (float)(1u << r.shift)) ++r.shift;
  if (r.shift > 8) r.floor = len * (float)kNaColsMost < kNaLeastWork ? kNaColsMost : (uint32_t)(kNaLeastWork / len);
  return r;
}
constexpr uint32_t na_cols(uint32_t k, uint32_t g, NaRuns r) {
  const uint32_t lo = na_columns(k, 0) >> r.shift, want = na_columns(k, g) >> r.shift;
  uint32_t n = lo < 4 ? 4 : (lo < 16 ? lo : (lo < r.floor ? lo : (r.floor < 16 ? 16 : r.floor)));
  if (n < want) n = want;
  if (n > kNaColsMost) n = kNaColsMost;
  return r.shift > 8 && n > 16 ? n & ~15u : n;
}
constexpr uint32_t na_items(uint32_t k, uint32_t g, uint32_t cols) { return (k - (64 * g + 1) + cols - 1) / cols; }
// Small families take the runs of one workgroup a CU in every class, and one
// launch; the most items any lengths give is na_runs_most's.
constexpr NaRuns na_runs_small() { return {8, 0}; }
constexpr NaRuns na_runs_most() { return {10, 0}; }
constexpr uint32_t na_all_items(uint32_t k, NaRuns r) {
  uint32_t n = 0;
  for (uint32_t g = 0; g < na_groups(k); ++g) n += na_items(k, g, na_cols(k, g, r));
  return n;
}

}  // namespace famsa
