// What the allocation-free call checks of its offsets before a residue is read
// (constant expressions, so that the kernel and the host run the same code).
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

}  // namespace famsa
