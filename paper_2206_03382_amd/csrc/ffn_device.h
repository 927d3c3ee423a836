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
// An expert's live tiles (row tiles below its fill x all column tiles) are numbered by blocks of 8 tile columns and, inside a block,
// row by row, so that 32 consecutive numbers are 4 row tiles x 8 column tiles that share A rows and B columns; the experts follow
// each other, and tile_number deals this sequence to the XCDs.  Every wave finds its tile by prefix sums over the experts, 64 to a
// step; no host has to know the fills.
template <int TILE_ROWS>
__device__ __forceinline__ bool find_tile(int b, int lane, int E, int64_t C, const int32_t* __restrict__ counts, int NT,
                                          int& e_out, int& mt_out, int& nt_out, int& rows_out) {
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
  const int t = tile_number(b, live);
  if (t < 0) return false;
#pragma unroll
  for (int c = 0; c < kChunks; ++c) {
    if (c * 64 >= E) break;
    const unsigned long long hit = __ballot(upto[c] > t);
    if (hit == 0) continue;
    const int l = __builtin_amdgcn_readfirstlane(__builtin_ctzll(hit));
    const int rows = __builtin_amdgcn_readlane(rowsv[c], l), mte = (rows + TILE_ROWS - 1) / TILE_ROWS;
    const int q = t - (__builtin_amdgcn_readlane(upto[c], l) - mte * NT);
    const int full = (NT / 8) * mte * 8;                            // its tiles in full 8-column blocks
    e_out = c * 64 + l;                                             // the same in every lane: in scalar registers
    rows_out = rows;
    if (q < full) {
      mt_out = (q % (mte * 8)) / 8;
      nt_out = (q / (mte * 8)) * 8 + q % 8;
    } else {
      const int w = NT % 8, r = q - full;
      mt_out = r / w;
      nt_out = (NT / 8) * 8 + r % w;
    }
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
