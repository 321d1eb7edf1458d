// The launch shape of a batch's staging, host arithmetic only.
#pragma once
#include <stdint.h>

namespace famsa {

// A workgroup stages a span of one sequence: every sequence has one, a long
// one as many more as its column stream needs (so that a sequence of 65,535
// residues is shared by 17 workgroups).  The spans past a sequence's first are
// listed, kStageSpan codes each, so short sequences beside a long one cost
// nothing more.
constexpr uint32_t kStageSpan = 4096;
constexpr uint32_t kStageThreads = 256;
// Workgroups at most: a launch holds fewer than 2^32 threads, and a workgroup
// takes further spans one after another.
constexpr uint32_t kStageMaxBlocks = 1u << 22;

// Codes of a sequence's column stream: whole chunks of 8 and one spare.
constexpr uint32_t stream_codes(uint32_t len) { return 8u * ((len + 7u) / 8u + 1u); }
// Spans past the first.
constexpr uint32_t stage_more_spans(uint32_t len) { return (stream_codes(len) - 1u) / kStageSpan; }
constexpr uint32_t stage_blocks(uint64_t spans) {
  return spans < kStageMaxBlocks ? (uint32_t)spans : kStageMaxBlocks;
}

struct StageSpan {
  uint32_t seq, span;  // codes span * kStageSpan on
};

}  // namespace famsa
