// What the grouped GEMM's kernels share: vector types, direct global->LDS loads, the tile search, a launch's arguments.
#pragma once
#include <cmath>
#include <type_traits>

#include "common.h"
#include "ffn_rules.h"

namespace moe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(8))) short short8v;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T*)(p))
#define PIN() __builtin_amdgcn_sched_barrier(0)

namespace {

// Direct global->LDS load of 16 bytes per lane from base + voff: lane l's data lands at lds_addr + 16 l.  Written as
// inline assembly so that the compiler does not serialise the prefetch against the LDS reads of the other stage;
// completion is tracked by hand (s_waitcnt vmcnt + barrier before a stage is read).
__device__ __forceinline__ void global_to_lds_16(const char* base, uint32_t voff, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %2\n\tglobal_load_lds_dwordx4 %0, %1" : : "v"(voff), "s"(base), "s"(lds_addr) : "memory", "m0");
}
// The same from an address of the lane's own; STREAM: with the nontemporal hint, for data that is read once.
template <bool STREAM = false> __device__ __forceinline__ void global_to_lds_16(const char* addr, uint32_t lds_addr) {
  if constexpr (STREAM) asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off nt" : : "v"(addr), "s"(lds_addr) : "memory", "m0");
  else asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" : : "v"(addr), "s"(lds_addr) : "memory", "m0");
}

// Inclusive prefix sum over the 64 lanes with data-parallel primitives (shifts inside rows of 16 lanes, then the rows'
// totals broadcast forward): no trip through the LDS crossbar, a few cycles per step.
__device__ __forceinline__ int wave_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);    // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);    // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);    // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);    // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15 into rows 1 and 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31 into rows 2 and 3
  return v;
}

}  // namespace

// Rows of expert e that exist: its fill, at most C.
__device__ __forceinline__ int live_rows_of(int e, int64_t C, const int32_t* __restrict__ counts) {
  if (!counts) return (int)C;
  const int64_t c = counts[e];
  return (int)(c < C ? (c > 0 ? c : 0) : C);
}

// Which tile block number b works on, or false where there is none for it.
// An expert's live tiles are its row tiles below the fill x all column tiles; how they are numbered and dealt to the XCDs: ffn_rules.h.  Every wave
// finds its tile by prefix sums over the experts, 64 to a step; no host has to know the fills.
// SHIFT: log2 of the blocks that share a unit, where groups are to hold as many more tiles.  SHORTS: short row tiles may come last.
template <int TILE_ROWS, int SHIFT, bool SHORTS, bool CUTS, int CHUNKS>
__device__ __forceinline__ bool search_tile(int b, int lane, int E, int64_t C, const int32_t* __restrict__ counts, int NT,
                                            int& e_out, int& mt_out, int& nt_out, int& rows_out, TileHalf& half) {
  int rowsv[CHUNKS], upto[CHUNKS], groups[CHUNKS];                  // lane l of chunk c: rows of expert 64 c + l; tall tiles, full groups of them up to it
  unsigned long long shortv[CHUNKS];                                // experts with a short row tile
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) rowsv[c] = c * 64 + lane < E ? live_rows_of(c * 64 + lane, C, counts) : 0;      // all loads in flight at once
  int tall = 0, shorts = 0;
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {                                // as if all row tiles were tall
    if (c > 0 && c * 64 >= E) break;
    upto[c] = tall + wave_inclusive_scan((rowsv[c] + TILE_ROWS - 1) / TILE_ROWS * NT);
    tall = __builtin_amdgcn_readlane(upto[c], 63);
  }
  bool apart = false;                                               // short row tiles come last
  if (SHORTS && counts && C > TILE_ROWS) {
    int all_rows = 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
      if (c > 0 && c * 64 >= E) break;
      all_rows += __builtin_amdgcn_readlane(wave_inclusive_scan(rowsv[c]), 63);
    }
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
      if (c > 0 && c * 64 >= E) break;
      apart |= __ballot(far_above_mean(rowsv[c], E, all_rows)) != 0;
    }
    if (apart || may_open_a_round(tall, SHIFT)) {
      int without = 0, upto_without[CHUNKS];
#pragma unroll
      for (int c = 0; c < CHUNKS; ++c) {
        if (c > 0 && c * 64 >= E) break;
        upto_without[c] = without + wave_inclusive_scan(tall_row_tiles(rowsv[c], TILE_ROWS, true) * NT);
        without = __builtin_amdgcn_readlane(upto_without[c], 63);
      }
      apart |= opens_a_round(without, tall, SHIFT);
      if (apart) {
        shorts = tall - without;
        tall = without;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
          if (c > 0 && c * 64 >= E) break;
          upto[c] = upto_without[c];
          shortv[c] = __ballot(rowsv[c] > tall_row_tiles(rowsv[c], TILE_ROWS, true) * TILE_ROWS);
        }
      }
    }
  }
  constexpr int gs = kGroupShift + SHIFT;
  int rounds = 0;
  if (deals_groups(tall, E, NT, SHIFT)) {
    int full = 0;
#pragma unroll
    for (int c = 0; c < CHUNKS; ++c) {
      if (c > 0 && c * 64 >= E) break;
      groups[c] = full + wave_inclusive_scan(tall_row_tiles(rowsv[c], TILE_ROWS, apart) * NT >> gs);
      full = __builtin_amdgcn_readlane(groups[c], 63);
    }
    rounds = full >> 3;
  }
  half = {-1, -1};
  if (CUTS && __builtin_expect(may_be_cut(b, gridDim.x, tall + shorts), 0) && !cut_tile(b, gridDim.x, tall, shorts, half)) return false;
  const TileSpot s = tile_spot(b, tall, shorts, rounds, gs);
  if (s.part == kNoTile) return false;
  int seen = 0;                                                     // short row tiles of earlier chunks
#pragma unroll
  for (int c = 0; c < CHUNKS; ++c) {
    if (c > 0 && c * 64 >= E) break;
    int inc = upto[c];                                              // groups, tiles that are left, or short tiles, up to this lane's expert
    if (rounds > 0) inc = s.part == kDealtTile ? groups[c] : inc - ((groups[c] < rounds * 8 ? groups[c] : rounds * 8) << gs);
    if (SHORTS && s.part == kShortTile) {
      const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(shortv[c] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)shortv[c], 0));
      inc = (seen + before + (int)(shortv[c] >> lane & 1)) * NT;
      seen += __builtin_popcountll(shortv[c]);
    }
    const unsigned long long hit = __ballot(inc > s.at);
    if (hit == 0) continue;
    const int l = __builtin_amdgcn_readfirstlane(__builtin_ctzll(hit));
    const int rows = __builtin_amdgcn_readlane(rowsv[c], l), mt = tall_row_tiles(rows, TILE_ROWS, apart), all = mt * NT;
    const int back = s.at - __builtin_amdgcn_readlane(inc, l);      // from the end of the expert's groups or tiles
    e_out = c * 64 + l;                                             // the same in every lane: in scalar registers
    rows_out = rows;
    if (SHORTS && s.part == kShortTile) {
      mt_out = mt;
      nt_out = NT + back;
    } else {
      const TileAt at = tile_in_expert(e_out, s.part == kDealtTile ? ((back + (all >> gs)) << gs) + (b / 8 & ((1 << gs) - 1)) : all + back, mt, NT);
      mt_out = at.mt;
      nt_out = at.nt;
    }
    return true;
  }
  return false;
}

// EQUAL: every expert has all of its C rows (weight gradients), see equal_tile.  Up to 64 experts, and up to 128, have code of their own, nearly one
// straight piece: what a launch of few tiles pays for is fetching it (decode step of 16 tokens 47.8 -> 46.9 us; second product of 128 experts x 8192 rows, 264
// tiles to a unit, 8150 -> 8080).
template <int TILE_ROWS, bool EQUAL = false, int SHIFT = 0, bool SHORTS = false, bool CUTS = false>
__device__ __forceinline__ bool find_tile(int b, int lane, int E, int64_t C, const int32_t* __restrict__ counts, int NT,
                                          int& e_out, int& mt_out, int& nt_out, int& rows_out, TileHalf& half) {
  if (EQUAL) {
    TileAt at;
    if (!equal_tile(b, E, (int)((C + TILE_ROWS - 1) / TILE_ROWS), NT, at)) return false;
    e_out = at.e;
    mt_out = at.mt;
    nt_out = at.nt;
    rows_out = (int)C;
    half = {-1, -1};
    return true;
  }
  if (E <= 64) return search_tile<TILE_ROWS, SHIFT, SHORTS, CUTS, 1>(b, lane, E, C, counts, NT, e_out, mt_out, nt_out, rows_out, half);
  if (E <= 128) return search_tile<TILE_ROWS, SHIFT, SHORTS, CUTS, 2>(b, lane, E, C, counts, NT, e_out, mt_out, nt_out, rows_out, half);
  return search_tile<TILE_ROWS, SHIFT, SHORTS, CUTS, kMaxExperts / 64>(b, lane, E, C, counts, NT, e_out, mt_out, nt_out, rows_out, half);
}

template <int TILE_ROWS, bool EQUAL = false, int SHIFT = 0, bool SHORTS = false>
__device__ __forceinline__ bool find_tile(int b, int lane, int E, int64_t C, const int32_t* __restrict__ counts, int NT,
                                          int& e_out, int& mt_out, int& nt_out, int& rows_out) {
  TileHalf half;
  return find_tile<TILE_ROWS, EQUAL, SHIFT, SHORTS>(b, lane, E, C, counts, NT, e_out, mt_out, nt_out, rows_out, half);
}

struct TileArgs {
  const void* A;
  const void* B;
  const void* bias;
  const int32_t* counts;
  const int32_t* gather;        // slot -> row [E, slots]: A is one matrix of gather_rows rows, [., K] (kNN) or [., C] (kTN, GK)
  int64_t gather_rows;
  int64_t C;                    // rows of A (kNN, kNT) or its width (kTN)
  int64_t K;                    // length of the reduction; slots per expert (kTN)
  int N, E, MT, NT;
  int plain;                    // block y, x = expert, tile of it; else the numbering of find_tile in x
  void* out;
  const int32_t* kfill;         // kTN: live slots per expert
  const void* pre;              // kNT: multiply by act'(pre) (act >= 0) or add pre (act < 0)
  void* pre_out;                // kNN: the values before the activation go here as well
  int act;                      // MOE_ACT_*, + kFullAct (bf16 results) for the form with erf and true divisions; < 0: none
  int64_t ktotal;               // PART: length of the whole reduction, of which every "expert" is K consecutive k
};

// Fills in the tile counts and the grid of a launch on tiles of bm x bn (total: rows of all experts that exist, at most); false
// where no grid holds it.
static inline bool tile_launch(TileArgs& p, int bm, int bn, int64_t total, dim3& grid) {
  p.MT = (int)ceil_div(p.C, bm);
  p.NT = (int)ceil_div(p.N, bn);
  // more experts than the search takes, or more blocks than a grid dimension holds (2^32 threads: launches beyond run cut short)
  int64_t blocks = tile_grid(p.NT, live_row_tiles(p.E, p.C, total, bm));
  p.plain = p.E > kMaxExperts || blocks >= kMaxBlocks;
  if (p.plain) blocks = (int64_t)p.MT * p.NT;
  grid = dim3((unsigned)blocks, p.plain ? (unsigned)p.E : 1);
  return blocks < kMaxBlocks;
}

// TileArgs::act of bf16 results: the form of the activations with erf and true divisions.
constexpr int kFullAct = 4;

namespace {

__device__ __align__(256) uint4 g_zero_piece[16];                   // stays zero: where pieces past the reduction's end are read

}  // namespace

}  // namespace moe
