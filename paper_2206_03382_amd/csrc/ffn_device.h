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
// An expert's live tiles (row tiles below its fill x all column tiles) are numbered as tile_in_expert says.  Hardware deals blocks
// round-robin, so block b runs on XCD b % 8, as the b / 8-th of its tiles, and the tiles that an XCD holds at one time should be neighbours
// in its own L2.  Launches of kDealtTiles tiles and more deal whole groups of 32 tiles of an expert to the XCDs in turn, in as many rounds as
// there are full ones for all eight.  Everything left (all of a smaller launch) is one sequence, expert by expert, cut into 8 runs of
// equal length (to a tile), one to an XCD: even whatever the fills are.  Groups of 8 to 32 tiles dealt throughout, short ones last,
// left XCDs with up to a round of tiles more than others: 17 experts x 14 tiles 42 us, 24 so; ViT layer of 32 experts x 784 rows 386 ->
// 353, training step of 17 x 353 rows 340 -> 309.  Runs of an eighth for every launch cost where XCDs next to each other
// share what they read beyond their L2: 8 experts x 4096 rows, 2048 x 2048 (1088 tiles) layer 592 us in groups, 604 in eighths, 603 in
// rounds of 32 cut without regard to experts, 0.996 of the rate in groups so; 17 x 353 (663 tiles) 328 in such rounds.  Experts of fewer than
// four row tiles on average have nothing for several XCDs to share and stay in eighths: 64 experts x 16 rows, 1024 x 4096 212.0 us
// dealt, 210.3 so.
// Every wave finds its tile by prefix sums over the experts, 64 to a step; no host has to know the fills.
constexpr int kDealtTiles = 1024;
// EQUAL: every expert has all of its C rows (weight gradients), see equal_tile.
template <int TILE_ROWS, bool EQUAL = false>
__device__ __forceinline__ bool find_tile(int b, int lane, int E, int64_t C, const int32_t* __restrict__ counts, int NT,
                                          int& e_out, int& mt_out, int& nt_out, int& rows_out) {
  if (EQUAL) {
    TileAt at;
    if (!equal_tile(b, E, (int)((C + TILE_ROWS - 1) / TILE_ROWS), NT, at)) return false;
    e_out = at.e;
    mt_out = at.mt;
    nt_out = at.nt;
    rows_out = (int)C;
    return true;
  }
  constexpr int kChunks = kMaxExperts / 64;
  int rowsv[kChunks], upto[kChunks];                                // lane l of chunk c: rows of expert 64 c + l; live tiles up to it
#pragma unroll
  for (int c = 0; c < kChunks; ++c) rowsv[c] = c * 64 + lane < E ? live_rows_of(c * 64 + lane, C, counts) : 0;      // all loads in flight at once
  int live = 0;                                                     // live tiles of all experts
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    if (c * 64 >= E) break;
    upto[c] = live + wave_inclusive_scan((rowsv[c] + TILE_ROWS - 1) / TILE_ROWS * NT);
    live = __builtin_amdgcn_readlane(upto[c], 63);
  }
  // tiles of expert l that are dealt in whole groups, and what of its tiles is left
  const int x = b % 8, i = b / 8;
  int rounds = 0, groups[kChunks];                                  // lane l of chunk c: full groups up to expert 64 c + l
  if (live >= kDealtTiles && live >= 4 * E * NT) {
    int full = 0;
#pragma unroll
    for (int c = 0; c < kChunks; ++c) {
      if (c * 64 >= E) break;
      groups[c] = full + wave_inclusive_scan(((rowsv[c] + TILE_ROWS - 1) / TILE_ROWS * NT) >> 5);
      full = __builtin_amdgcn_readlane(groups[c], 63);
    }
    rounds = full >> 3;
  }
  const bool dealt = i < rounds * 32;
  const int left = live - rounds * 256;
  const int target = dealt ? (i >> 5) * 8 + x : x * left / 8 + i - rounds * 32;
  if (!dealt && target >= (x + 1) * left / 8) return false;
  int seen = 0;
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    if (c * 64 >= E) break;
    const int tiles = (rowsv[c] + TILE_ROWS - 1) / TILE_ROWS * NT;
    int mine = 0, inc;                                              // dealt groups of this lane's expert
    if (rounds > 0) {
      const int before = groups[c] - (tiles >> 5), most = rounds * 8 - before;
      mine = most < 0 ? 0 : (most < tiles >> 5 ? most : tiles >> 5);
    }
    if (dealt) inc = groups[c];
    else inc = rounds > 0 ? seen + wave_inclusive_scan(tiles - 32 * mine) : upto[c];
    const unsigned long long hit = __ballot(inc > target);
    if (hit == 0) { seen = __builtin_amdgcn_readlane(inc, 63); continue; }
    const int l = __builtin_amdgcn_readfirstlane(__builtin_ctzll(hit));
    const int rows = __builtin_amdgcn_readlane(rowsv[c], l), mte = (rows + TILE_ROWS - 1) / TILE_ROWS;
    const int in = __builtin_amdgcn_readlane(inc, l), all = mte * NT, gone = __builtin_amdgcn_readlane(mine, l);
    const int q = dealt ? (target - (in - (all >> 5))) * 32 + (i & 31) : 32 * gone + target - (in - (all - 32 * gone));
    const TileAt at = tile_in_expert(c * 64 + l, q, mte, NT);
    e_out = at.e;                                                   // the same in every lane: in scalar registers
    mt_out = at.mt;
    nt_out = at.nt;
    rows_out = rows;
    return true;
  }
  return false;
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
  int64_t blocks = tile_grid(p.E, p.MT, p.NT, live_row_tiles(p.E, p.C, total, bm));
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
