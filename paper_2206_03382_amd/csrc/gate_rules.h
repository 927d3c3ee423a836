// Which form of the gate's kernels a call takes: plain host arithmetic on sizes, kept apart from the kernels so that a test can
// ask it without a GPU.
#pragma once
#include <stdint.h>

namespace moe {

// Whether the arrivals are scanned and the slots assigned in one launch (gate_slots_kernel, whose every block adds up all counters
// by itself) instead of two.  Measured in captured graphs with the top-k, one launch against two: 2048 tokens, 8 experts, top-2
// (512 counters) 7.4 and 8.8 us; at 1024 counters 7.6 and 7.9 (8192 tokens, 8 experts, top-1), 9.2 and 9.8 (1024 tokens, 32,
// top-2); at 2048 9.4 and 8.0 (16384, 8, top-1), 10.7 and 9.8 (4096, 16, top-2); at 4096 13.5 and 9.4 (16384, 8, top-2), 18.4 and
// 8.8 (32768, 8, top-1).  Many (expert, rank) pairs, and more experts than the few blocks can mark unfilled slots for, cost as
// well: 64 tokens, 32 experts 8.8 and 7.6; 256 tokens, 64 experts, top-4 13.7 and 12.9.
constexpr int kSlotsMaxCounters = 1024, kSlotsMaxPairs = 128;
inline bool slots_in_one_launch(int64_t token_blocks, int64_t E, int k) {
  return E * k <= kSlotsMaxPairs && E * k * token_blocks <= kSlotsMaxCounters && E <= 16 * token_blocks;
}

// Tokens to a block of gate_dx_kernel.  Every block reads the whole of Wg: few tokens to a block spread a small launch over the
// chip, many keep those reads down.  Measured with 4 and with 16, fp32, dx alone: 1024 tokens, M = 2048, 17 experts 31.3 and
// 20.5 us, 4096, 2048, 300 1658 and 457; 256, 2048, 17 15.4 and 17.8; 2048, 776, 24 15.5 and 16.4; 4096, 776, 24 24.0 and 17.9;
// bf16 4096, 2048, 17 30.1 and 23.5, 1024, 2048, 17 12.3 and 16.0.  The two meet near 8 MB of tokens whatever the width and the type.
inline int gate_dx_tokens(int64_t T, int64_t row_bytes) { return T * row_bytes >= 8000000 ? 16 : 4; }

}  // namespace moe
