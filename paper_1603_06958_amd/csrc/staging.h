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

// Bytes that a sequence's codes take in the batch.  The plain kernel reads them,
// a byte a step and lane, 64 columns in a wave: its plans start every sequence
// at 32 bytes (100,000 sequences of 261: 12.40 s a pass, back to back 13.75;
// 10,000 of 300 the same either way).  For other plans only the staging reads
// them, and they lie as the caller's do, one copy.
constexpr uint64_t code_bytes(uint32_t len, bool spaced) { return spaced ? (len + 31ull) / 32ull * 32ull : len; }

struct StageSpan {
  uint32_t seq, span;  // codes span * kStageSpan on
};

}  // namespace famsa
