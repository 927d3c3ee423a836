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

// Whether top-k, scan and assignment all run in one block (gate_small_kernel: a lane per token, its logits in registers).  marked_C:
// slots per expert that have to be marked unfilled, which one block does slowly where they are many; 0 if none are.  Measured in captured
// graphs, two or three launches and this one: 64 tokens, 3 experts, top-3 6.2 and 4.3 us, 256, 16, 2 7.5 and 5.1, 512, 8, 4 8.0
// and 5.7, 1024, 16, 1 6.5 and 5.8, 1024, 8, 4 8.6 and 8.6.  Many ranks are its serial part: 64, 16, 4 10.1 and 10.5, 1024, 16, 8 16.5 and
// 23.4.  Rows that are not a power of two long come value by value, which many waves on one unit do slowly: 24, 6, 2 5.9 and 4.6, 64,
// 5, 5 8.2 and 7.1, but 1000, 13, 1 6.3 and 8.3.
constexpr int kSmallGateTokens = 1024, kSmallGatePairs = 32;
inline bool gate_in_one_block(int64_t T, int64_t E, int k, int64_t marked_C) {
  return T <= ((E & (E - 1)) == 0 ? kSmallGateTokens : 256) && E <= 16 && E * k <= kSmallGatePairs && E * marked_C <= 16 * kSmallGateTokens;
}

// Whether such a gate's logits are computed by that block as well (gate_few_tokens_kernel): where they are one tile of 16 tokens x 16 experts, which one block
// computes anyhow.  (More tokens are more tiles, which as many units compute at once.)  One or two experts, which have lane groups of
// their own in the decisions, would need two more instantiations per type, for gates that leave little to choose: they stay with two launches.
constexpr int64_t kFewGateTokens = 16;
inline bool gate_of_few_tokens(int64_t T, int64_t E, int k, int64_t marked_C) {
  return T <= kFewGateTokens && E > 2 && gate_in_one_block(T, E, k, marked_C);
}

// Blocks of 64 tokens from which wide gates decide with one lane per token (M: length of the products that repair near-ties; 0: none are
// repaired).  Below, a token's lane group spreads a block's work over more of the chip: 6000 tokens, 64 experts, top-4: 19 us against 23 (51 against 73
// with repairs); 65536 tokens, top-2: 27 against 21.  At the line itself (32768 tokens) the two are alike for up to four choices (top-1 of
// 32 12.4 and 11.0 us, top-4 of 64 24.1 and 23.3).  More choices have more near-ties, and a lane's repairs are a wave's serial
// part, so with repairs the line lies further out, the longer a product is.  Whole gates with top-5 and top-8 of 24 to 256 experts, 32768 to 65472 tokens,
// group and lane: 32768 tokens, M = 4096, top-8 of 128 170 and 264 us; M = 1024, top-8 of 64 95 and 117; 49152, M = 4096, top-8 of 256 491 and 558;
// 65472, M = 4096, top-8 of 64 292 and 318, but M = 1024 165 and 152, M = 512, top-8 of 256 1.20 times as long in groups; of 32 experts 40000, M = 1024 108 and 91.
// Over 260 such gates this line is 0.4 % off the better form on average (10 % at most), 512 for all 6.8 %, 768 and 1024 by the number of experts 3.8 %.
// Without repairs 512 is 3.2 % off over 92 gates and 768 and 1024 20 %: lanes are the faster from there on for nearly all (top-8 of 160 92 and
// 64 us, 65472 tokens 172 and 79; top-5 of 24 38 and 28), though not for a few choices of many experts (32768 tokens, top-5 of 128 32 and
// 46, of 512 87 and 141).
inline int64_t gate_lane_topk_blocks(int64_t E, int k, int64_t M) {
  if (k <= 4 || M == 0) return 512;
  const int64_t line = E <= 32 ? 256 + M / 8 : 448 + M / 6;
  return line < 512 ? 512 : (line > 1024 ? 1024 : line);
}

// Experts whose exact logits the wide kernel takes (vecw: its 16-byte pieces of Wg's rows are whole): whole 128s, two of its blocks, and what is left
// beyond them if it is more than 96; the narrow kernel takes the others, 64 at a time.  A block's 64 columns take the same time whether they are filled or not, and few
// tokens leave units without a block.  fp32, M = 2048, all narrow and all wide: 4096 tokens, 128 experts 54 and 75 us, 16384 168 and 175, 32768 324 and 319, 65536 658 and
// 610; 12000, 512 486 and 455; 65536, 72 468 and 602, 96 517 and 604, 104 688 and 605, 120 686 and 609; 136 722 as 128 + 8, 792 and 880; 160 774 as 128 + 32, 837 and 876.
// Only at 64 beyond a 128 all wide would be the better: 192 936 as 128 + 64, 983 and 890 (32768 tokens 489, 486 and 463).
inline int64_t gate_logits_wide_experts(int64_t T, int64_t E, bool vecw) {
  if (E <= 64 || !vecw || T * E < ((int64_t)1 << 22)) return 0;
  const int64_t left = E % 128;
  return left <= 96 ? E - left : E;
}

// Lanes to a token and tokens to a block of gate_backward_kernel, whose blocks walk rounds of 256 / lanes tokens, one behind the
// other.  Few tokens take one round; with dbias, whose rows of one per block are added up in another launch, many take more.
// Measured with 1, 2 and 4 rounds: without dbias 8192 tokens, 8 experts 4.4, 5.2 and 7.2 us, 65536 6.1, 6.2 and 7.7, 131072, 64 experts
// 27.7, 27.5 and 29.6; with it 8192, 8 8.0, 8.6 and 11.1, 32768, 32 20.2, 15.1 and 15.6, 65536, 32 35.1, 24.8 and 20.5.
inline int gate_backward_lanes(int64_t E) { return E <= 8 ? 8 : (E <= 128 ? 16 : 64); }
inline int64_t gate_backward_token_block(int64_t T, int64_t E, bool bias) {
  const int64_t tokens = 256 / gate_backward_lanes(E);
  int64_t rounds = T < 8192 ? 1 : (T < 65536 ? (bias ? 2 : 1) : (bias ? 4 : 2));
  while ((T + tokens * rounds - 1) / (tokens * rounds) >= ((int64_t)1 << 24)) rounds *= 2;   // a grid dimension holds fewer than 2^32 threads
  return tokens * rounds;
}

// Tokens to a block of gate_dx_kernel.  Every block reads the whole of Wg: few tokens to a block spread a small launch over the
// chip, many keep those reads down.  Measured with 4 and with 16, fp32, dx alone: 1024 tokens, M = 2048, 17 experts 31.3 and
// 20.5 us, 4096, 2048, 300 1658 and 457; 256, 2048, 17 15.4 and 17.8; 2048, 776, 24 15.5 and 16.4; 4096, 776, 24 24.0 and 17.9;
// bf16 4096, 2048, 17 30.1 and 23.5, 1024, 2048, 17 12.3 and 16.0.  The two meet near 8 MB of tokens whatever the width and the type:
// 8.4 MB, fp32, 4096, 512, 8 10.3 and 10.8, 4096, 512, 64 32.4 and 27.1; 16.8 MB, 8192, 512, 8 14.4 and 12.7.
inline int gate_dx_tokens(int64_t T, int64_t row_bytes) { return T * row_bytes >= 8000000 ? 16 : 4; }

}  // namespace moe
