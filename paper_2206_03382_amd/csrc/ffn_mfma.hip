// Grouped bf16 GEMM on the gfx950 matrix cores for the local experts' feed-forward layer
// (arXiv 2206.03382 Sec. 2.1; one [C, K] slab per expert, the layout of Sec. 4.2 "Flexible All-to-All").
//
//   out[e] = epilogue(A[e] (rows_e x K) * B[e] (K x N) + bias[e]),  A [E,C,K], B [E,K,N], out [E,C,N], all bf16,
//   fp32 accumulation, rows_e = min(counts[e], C) (or C).  Requires K % 64 == 0 and N % 256 == 0.
//
// Tiling: one 256-thread block (4 waves, one per SIMD) owns a 256 x 256 output tile; waves form a 2 x 2 grid, each
// owning 128 x 128 as 8 x 8 tiles of v_mfma_f32_16x16x32_bf16 (256 accumulator registers per lane).  Large wave tiles
// keep LDS->register traffic, the scarce resource on this chip, at 2 x 128 x 2 bytes per k per wave.  K advances in
// steps of 64 through LDS rings of two stages for A and three for B (5 x 32 KB, all of a unit's LDS) filled by direct global->LDS
// loads (16 bytes per lane, no staging registers).  Within a wave every MFMA is followed by at most one LDS read and one direct load, so the
// data movement of the next sub-step hides in the shadow of the current sub-step's MFMAs; one workgroup barrier per
// K-step hands the LDS stages over.
//
// What bounds it is the board's power limit, and next to it the way from L2 into LDS.  4 x 4 tiles of v_mfma_f32_32x32x16_bf16 take
// more power for the same product; on the same two stages of each operand 8192^3 (two products) took 1528 us so and 1448 in this form, 8
// experts x 4096 rows, 2048 x 2048 483 and 467, 32 x 8192, 4096 x 1024 3994 and 3857.  With two stages of each operand all sixteen
// loads of a K-step crowd into the half of a K-step between the barrier that frees their stage and its end.  The third stage of B
// lets its loads go out before the barrier and A's after it, one in 6 to 8 products throughout: the same shapes, on another board,
// 1496 -> 1467 us, 475 -> 446, 3865 -> 3604 (1.5, 1.23 and 1.22 PFLOP/s; a tile of 16 to 64 K-steps spends 8 to 10 us outside the loop).  By counters, 128 experts x 8192 rows, 4096 x 1024, before
// both and now: matrix cores busy 0.68 -> 0.71 of the time at 1.60 -> 1.64 GHz, and 0.51 -> 0.54 at 1.82 -> 1.89 in the
// second product.  Weight gradients with few K-steps or few tiles per unit, which the power limit does not bind, were up to 8 %
// faster on the former loop (16 experts x 495 slots, 1536 x 3072: 104 and 109 us), the others are up to 14 % faster on this one.
//
// LDS layouts (both written by the direct loads, which place lane l's 16 bytes at base + 16 l):
//   A tile  [256 rows][8 chunks of 8 k]:   chunk g of row r is stored at chunk position g ^ ((r / 2) % 8), so the 16 lanes
//           that share an LDS cycle of a ds_read_b128 (16 consecutive rows, same g) cover all 64 banks once.
//   B tile  [64 k][32 chunks of 8 n]:      chunk c of row k is stored at position c ^ (4 (k % 4)) ^ (2 (k / 8 % 2)); the two
//           16-lane blocks of a ds_read_b64_tr_b16 that share a cycle (4 k rows x 32 bytes each, 8 k apart) then cover all
//           banks once.
// B is K x N with N contiguous, but the matrix cores want k-contiguous operands: ds_read_b64_tr_b16 transposes
// 4 k x 16 n sub-blocks on the way out of LDS (source lane s of a 16-lane block supplies row k0 + s/4,
// columns n0 + 4 (s%4) .. +3; result lane l holds column n0 + l, rows k0 .. k0+3).
//
// Operand layouts (MODE).  The forward products read A row-major with k contiguous and B row-major with n contiguous
// (kNN).  The backward needs the other two combinations and gets them without any transposed copy in memory:
//   kNT: B is given as [N, K] (k contiguous, e.g. a weight matrix used transposed): its tile is staged and read
//        exactly like an A tile ([256 n][8 chunks of 8 k], ds_read_b128);
//   kTN: A is given as [K, rows] (rows contiguous, e.g. activations used transposed for a weight gradient): its tile
//        is staged and read exactly like a B tile ([64 k][32 chunks of 8 m], transposing reads).  Here the reduction
//        runs over an expert's slots, so its length differs per expert: K-steps up to the last whole one come from
//        the operands themselves and the last one from two small side buffers [E, 64, rows] / [E, 64, N] that hold
//        the remaining slots followed by zeros (written by tail_rows_kernel below), so no read ever touches a slot
//        past the fill.
//
// The two MFMA operands are passed swapped (B fragment first), so that a lane's accumulator registers hold four
// consecutive output columns of one row: D'[n][m] with m = lane % 16, n = 4 (lane/16) + v.  The
// epilogue packs them to 8 bytes, transposes the wave's 128 x 128 tile through LDS and stores whole 256-byte row pieces.
#include "ffn_device.h"

namespace moe {

namespace {

constexpr int BM = kLargeTile, BN = kLargeTile, BK = kLargeK;
constexpr int kThreads = 256;
constexpr int kTileBytes = 32768;           // one K-step of A, or of B
constexpr int kBRing = 2 * kTileBytes;      // LDS: two stages of A, then three of B
constexpr int kRingBytes = 5 * kTileBytes;
// Schedule of a K-step's 128 products per wave: the LDS reads of the next sub-step spread over a sub-step's first 48 products,
// B's eight direct loads of the K-step after next behind every sixth product up to the barrier, which is behind the 57th, and A's
// behind every eighth from there on.  All sixteen behind the barrier, every fourth product: 2-5 % slower, with or without the third stage
// of B loaded a K-step further ahead; A's behind every fourth or sixth product: up to 1 %; reads over 40 or 56 products and the barrier
// moved with them: 1-2 %.  With gathered rows of a transposed A both operands' loads stay behind the barrier, because the wait for
// the row indices ahead of it would wait for B's as well: sixteen behind every fourth product, A's first.  (A's behind every eighth and B's
// between their second half: 3 % slower over 16 weight gradients, 128 experts x 2048 rows, 4096 x 1024 2235 -> 2136 us.)
constexpr int kReadSpan = 48, kBarrierAt = 56, kLoadEveryA = 8, kLoadEveryB = 6, kLoadEveryGathered = 4;

// Branch-free activations for the bf16 epilogue.  gelu(v) = v Phi(v) with Phi(-y) = erfc(y / sqrt 2) / 2 for y = |v|:
// e = 2^-P(y) with a degree-5 polynomial P fitted to -log2 erfc(y / sqrt 2) (weighted least squares on [0, 9] with P(0) = 0;
// |gelu error| < 6e-7 everywhere, three orders below bf16 resolution), then Phi = 1 - e/2 for
// v >= 0 and e/2 for v < 0.  One exponential, no division.
constexpr float kGeluC1 = 1.151000500e+00f, kGeluC2 = 4.595958591e-01f, kGeluC3 = 5.214662850e-02f,
                kGeluC4 = -7.198722102e-03f, kGeluC5 = 4.881033092e-04f;
__device__ __forceinline__ float fast_gelu(float v) {
  const float y = fabsf(v);
  float p = fmaf(kGeluC5, y, kGeluC4);
  p = fmaf(p, y, kGeluC3);
  p = fmaf(p, y, kGeluC2);
  p = fmaf(p, y, kGeluC1);
  const float e = __builtin_amdgcn_exp2f(-(p * y));
  const float d = copysignf(fmaf(-0.5f, e, 0.5f), v);              // Phi(v) - 1/2
  return v * (0.5f + d);
}

// gelu'(v) = Phi(v) + v phi(v) with the same Phi and phi(v) = exp2(-v^2 / (2 ln 2)) / sqrt(2 pi): two exponentials,
// |error| < 3e-6.
constexpr float kHalfLog2e = 0.72134752f, kInvSqrt2Pi = 0.39894228f;
__device__ __forceinline__ float fast_gelu_grad(float v) {
  const float y = fabsf(v);
  float p = fmaf(kGeluC5, y, kGeluC4);
  p = fmaf(p, y, kGeluC3);
  p = fmaf(p, y, kGeluC2);
  p = fmaf(p, y, kGeluC1);
  const float e = __builtin_amdgcn_exp2f(-(p * y));
  const float d = copysignf(fmaf(-0.5f, e, 0.5f), v);              // Phi(v) - 1/2
  const float dens = __builtin_amdgcn_exp2f(-kHalfLog2e * v * v) * kInvSqrt2Pi;
  return fmaf(v, dens, 0.5f + d);
}

// act'(p) for the epilogue that turns dH into dP (bf16 results: relative error far below the output resolution)
template <int ACT> __device__ __forceinline__ float epilogue_act_grad(float p) {
  if (ACT == MOE_ACT_RELU) return p > 0.f ? 1.f : 0.f;
  if (ACT == MOE_ACT_GELU) return fast_gelu_grad(p);
  const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-p));        // SiLU
  return sg * fmaf(p, 1.f - sg, 1.f);
}

template <int ACT> __device__ __forceinline__ float epilogue_act(float v) {
  if (ACT == MOE_ACT_RELU) return fmaxf(v, 0.f);
  if (ACT == MOE_ACT_GELU) return fast_gelu(v);
  if (ACT == MOE_ACT_SILU) return v * __builtin_amdgcn_rcpf(1.0f + __expf(-v));
  return v;
}

// The activations of bf16 results.  The fit behind epilogue_act is good to 6e-7, which is below a bf16 rounding except where GeLU
// itself is small: at -4 it is off by 0.4 %, twice that rounding, and the erf form by 0.02 %.  Widths the large tile does not
// take have always had the erf form (and true divisions) and keep it, whichever tile they run on; widths it takes keep the fit.
template <int ACT> __device__ __forceinline__ float tile_act(float v) {
  if constexpr (ACT >= kFullAct) return apply_act(v, ACT - kFullAct);
  else return epilogue_act<ACT>(v);
}
template <int ACT> __device__ __forceinline__ float tile_act_grad(float p) {
  if constexpr (ACT >= kFullAct) return apply_act_grad(p, ACT - kFullAct);
  else return epilogue_act_grad<ACT>(p);
}

struct Frags {
  bf16x8 a[8], b[8];
};

}  // namespace

#include "ffn_ring.h"
#include "ffn_tile.h"
#include "ffn_half.h"
#include "ffn_piece.h"


// ---- main loop -------------------------------------------------------------------------------------------------
// K-step kt (64 wide) is two sub-steps of 64 MFMAs.  While sub-step s computes from one fragment buffer, the LDS reads of
// sub-step s+1 (24, or 16 / 32 with no / two transposed operands) fill the other.  The direct loads of K-step kt+2 fill stages that
// an earlier K-step was read from: B's that of kt-1, so they go out from the start of K-step kt; A's that of kt itself, so they
// start only behind the barrier that follows the last read of that stage, near the end of sub-step 0.  The barrier of K-step kt+1
// waits for both, but not for the eight of B's kt+3 that are behind them by then.
// GK (kTN only): the k-rows of A are gathered.  K-step t's row 2 (4 q + wave) + kg is row gk.rows[64 t + ...] of the
// matrix at a_base (row length gk.row_bytes); a_voff[0] then holds the lane's offset into the side buffer for q = 0.
struct GatherK {
  const int32_t* rows;          // this expert's slot -> row map (uniform)
  uint32_t row_bytes;           // bytes per row of the gathered matrix
  uint32_t nrows;               // rows of the gathered matrix (indices outside read row 0)
  uint32_t col;                 // per lane: byte offset of its 16-byte piece inside a row, for even q (odd q: the swizzle's 2 (k / 8 % 2), 32 bytes)
  uint32_t tail_step;           // bytes between the side buffer's k-rows of consecutive q
};
// FAR: A's rows lie up to 64 GiB apart (gathered from a token matrix beyond 4 GiB): offsets count 16-byte pieces, and a load takes
// a 64-bit address of the lane's own, formed beside the matrix instructions.  Without it such layers ran on the 128 x 128 tile:
// 2^19 tokens, M = H = 4096, 8 experts, layer 35.8 ms, 30.8 with it; training step 112.0, 96.1.
template <int NI, int MODE, bool GK = false, bool FAR = false>
__device__ __forceinline__ void tile_main_loop(char* smem, const char* a_base, const char* b_base, const char* a_last,
                                               const char* b_last, const uint32_t (&a_voff)[8],
                                               const uint32_t (&b_voff)[8], int64_t a_step, int64_t b_step,
                                               const int (&a_off)[8], const int (&b_off)[8], int kg, int kq,
                                               int a_mask, int wave, int KT, const uint16_t* bias_w,
                                               f32x4 (&acc)[8][8], const GatherK& gk = GatherK{}) {
  constexpr bool FULL = NI == 4;
  constexpr bool TRA = MODE == kTN;          // A through transposing reads (two per fragment)
  constexpr bool TRB = MODE != kNT;          // B through transposing reads
  constexpr int NRA = TRA ? 16 : 8, NRB = TRB ? 16 : 8, NR = NRA + NRB;   // LDS reads per sub-step
  constexpr int PA = TRA ? 2 : 1;
  Frags f[2];
  const uint32_t smem_addr = (uint32_t)(uintptr_t)LDS_PTR(char, smem);

  // read number r (0 .. NR-1) of sub-step s (32 k) from `stage` into fragment buffer `d`: the first of A, then B's, then the
  // rest of A's, the order in which the products want them.  A direct read fetches a lane's 8 k of one row (ds_read_b128; off[s]
  // is the lane's address of sub-tile 0); a transposed fragment takes two reads of 4 k each (off[t] is sub-tile t's address).
  auto read_direct = [&](const char* stage, const int (&off)[8], int t, int s) -> bf16x8 {
    return *LDS_PTR(bf16x8, stage + off[s] + t * 2048);
  };
  auto read_tr = [&](const char* stage, const int (&off)[8], int t, int s, int half) -> short4v {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4v, stage + off[t] + (32 * s + 4 * half) * 512));
  };
  auto join = [](short4v lo, short4v hi) -> bf16x8 {
    return __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto read = [&](const char* a_stage, const char* b_stage, int s, int r, Frags& d, short4v& lo) {
    const bool is_b = r >= PA && r < PA + NRB;
    if (is_b) {
      const int rb = r - PA;
      if (NI > 0) {
        if (!TRB) d.b[rb] = read_direct(b_stage, b_off, rb, s);
        else if ((rb & 1) == 0) lo = read_tr(b_stage, b_off, rb >> 1, s, 0);
        else d.b[rb >> 1] = join(lo, read_tr(b_stage, b_off, rb >> 1, s, 1));
      }
    } else {
      const int ra = r < PA ? r : r - NRB;
      if (!TRA) { if (ra < 2 * NI) d.a[ra] = read_direct(a_stage, a_off, ra, s); }
      else if ((ra & 1) == 0) lo = read_tr(a_stage, a_off, ra >> 1, s, 0);
      else d.a[ra >> 1] = join(lo, read_tr(a_stage, a_off, ra >> 1, s, 1));
    }
  };
  // direct load number idx (0..15: A0..A7, B0..B7) of K-step `tile` (the caller guarantees tile < KT).  With a
  // transposed A the last K-step comes from the zero-padded side buffers.
  // gathered A: the eight row indices of one K-step are fetched a K-step before they are needed (plain loads, so the
  // wait the compiler puts before their use falls behind the barrier's own wait) and turned into offsets in place.
  // The last K-step comes from the zero-padded side buffer instead (tail).
  auto gather_fetch = [&](int tile, uint32_t (&g)[8]) {
    const int32_t* p = gk.rows + (int64_t)tile * BK + wave * 2 + kg;
#pragma unroll
    for (int q = 0; q < 8; ++q) g[q] = (uint32_t)p[8 * q];
  };
  auto gather_offsets = [&](bool tail, uint32_t (&g)[8]) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (tail) {
        g[q] = ((a_voff[0] ^ (32 * (q & 1))) + q * gk.tail_step) >> (FAR ? 4 : 0);
      } else {
        const uint32_t r = g[q] < gk.nrows ? g[q] : 0u;
        g[q] = r * (gk.row_bytes >> (FAR ? 4 : 0)) + ((gk.col ^ (32 * (q & 1))) >> (FAR ? 4 : 0));
      }
    }
  };
  auto load_a = [&](const char* base, uint32_t off, uint32_t dst) {
    if constexpr (FAR) global_to_lds_16(base + ((uint64_t)off << 4), dst);
    else global_to_lds_16(base, off, dst);
  };
  uint32_t gv[8];
  auto dma_a = [&](int q, int tile) {
    const uint32_t dst = smem_addr + (tile & 1) * kTileBytes + (q * 4 + wave) * 1024;
    const bool last = MODE == kTN && tile == KT - 1;
    if (GK) {
      load_a(last ? a_last : a_base, gv[q], dst);
    } else {
      const char* src = last ? a_last : a_base + tile * a_step;
      if (FULL || ((a_mask >> q) & 1)) load_a(src, a_voff[q], dst);     // skip rows past the slab's fill
    }
  };
  // b_src is the K-step of B that the next loads take
  const char* b_src = MODE == kTN && KT == 1 ? b_last : b_base;
  auto dma_b = [&](int q, int stage) {                              // stage: byte offset in B's ring
    global_to_lds_16(b_src, b_voff[q], smem_addr + kBRing + stage + (q * 4 + wave) * 1024);
  };
  auto b_advance = [&](int tile) {
    if (MODE == kTN) b_src = tile < KT - 1 ? b_src + b_step : b_last;
    else b_src += b_step;
  };
  auto mfma = [&](int m, const Frags& c) {
    const int i = m >> 3, j = m & 7;
    if (i < 2 * NI) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c.b[j], c.a[i], acc[i][j], 0, 0, 0);
  };
  // One K-step; DMA: a K-step kt+2 exists; NEXT: a K-step kt+1 exists, or the reads ahead find a stage that holds nothing new and
  // are not used.  Every body more makes the compiler move accumulators around between them (with two transposed operands every
  // one less makes it spill).
  int b_stage = 0;                                                  // byte offset of K-step kt's stage in B's ring
  auto kstep = [&](auto dma_tag, auto next_tag, int kt, auto tail_tag) __attribute__((always_inline)) {
    constexpr bool DMA = decltype(dma_tag)::value, NEXT = decltype(next_tag)::value;
    const char* a_cur = smem + (kt & 1) * kTileBytes;
    const char* a_nxt = smem + (~kt & 1) * kTileBytes;
    const int b_fill = b_stage == 0 ? 2 * kTileBytes : b_stage - kTileBytes;   // of K-step kt-1 before, of kt+2 now
    const char* b_cur = smem + b_stage;
    b_stage = b_stage == 2 * kTileBytes ? 0 : b_stage + kTileBytes;
    const char* b_nxt = smem + b_stage;
    constexpr bool tail = decltype(tail_tag)::value;                // gathered A: K-step kt+2 is the last one
    if (GK && DMA && !tail) { gather_fetch(kt + 2, gv); PIN(); }
    short4v lo;
    auto read_at = [&](int m) { const int r = (m * NR + kReadSpan - 1) / kReadSpan; return r < ((m + 1) * NR + kReadSpan - 1) / kReadSpan ? r : NR; };
    auto loads = [&](int m) {                                       // m: products of this K-step so far
      if (!DMA) return;
      const int p = m - kBarrierAt;
      if (GK) {
        const int n = p >= 0 && p % kLoadEveryGathered == 1 ? p / kLoadEveryGathered : 16;
        if (n < 8) dma_a(n, kt + 2);
        else if (n < 16) dma_b(n - 8, b_fill);
        return;
      }
      if (m % kLoadEveryB == 1 && m / kLoadEveryB < 8) dma_b(m / kLoadEveryB, b_fill);
      if (p >= 0 && p % kLoadEveryA == 1 && p / kLoadEveryA < 8) dma_a(p / kLoadEveryA, kt + 2);
    };
#pragma unroll
    for (int m = 0; m < 64; ++m) {
      mfma(m, f[0]);
      PIN();
      if (const int r = read_at(m); r < NR) read(a_cur, b_cur, 1, r, f[1], lo);
      if (m == kBarrierAt) {
        // K-step kt+1 has landed, though not B's eight loads of kt+2 behind it; reads of this K-step are done
        if (DMA && !GK) asm volatile("s_waitcnt vmcnt(8) lgkmcnt(0)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
        PIN();
        asm volatile("s_barrier" ::: "memory");
        PIN();
        if (GK && DMA) { gather_offsets(tail, gv); PIN(); }          // nothing else is in flight here
      }
      loads(m);
      PIN();
    }
#pragma unroll
    for (int m = 0; m < 64; ++m) {
      mfma(m, f[1]);
      PIN();
      if (const int r = read_at(m); NEXT && r < NR) read(a_nxt, b_nxt, 0, r, f[0], lo);
      loads(m + 64);
      PIN();
    }
    if (DMA) b_advance(kt + 3);
  };

  uint32_t gv1[8];
  if (GK) {                                                         // both K-steps' indices before any direct load is in flight
    if (KT > 1) gather_fetch(0, gv);
    if (KT > 2) gather_fetch(1, gv1);
    gather_offsets(KT == 1, gv);
  }
#pragma unroll
  for (int q = 0; q < 8; ++q) dma_a(q, 0);
#pragma unroll
  for (int q = 0; q < 8; ++q) dma_b(q, 0);
  b_advance(1);
  if (KT > 1) {
    if (GK) {
      gather_offsets(KT == 2, gv1);
#pragma unroll
      for (int q = 0; q < 8; ++q) gv[q] = gv1[q];
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) dma_a(q, 1);
#pragma unroll
    for (int q = 0; q < 8; ++q) dma_b(q, kTileBytes);
    b_advance(2);
  }
  // while the first stages are in flight: the accumulators start from the bias (register u of tile (i, j) is column
  // 16 j + 4 kq + u of the wave's 128), or from zero
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (bias_w) {
      const u32x2 bb = *reinterpret_cast<const u32x2*>(bias_w + j * 16 + 4 * kq);
      b = f32x4{__uint_as_float(bb.x << 16), __uint_as_float(bb.x & 0xffff0000u), __uint_as_float(bb.y << 16), __uint_as_float(bb.y & 0xffff0000u)};
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) if (i < 2 * NI) acc[i][j] = b;
  }
  PIN();
  if (KT > 1) {
    if (FULL) asm volatile("s_waitcnt vmcnt(16)" ::: "memory");     // loads return in order: K-step 0 has landed
    else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");           // ragged tiles issue fewer loads of A: wait for both K-steps'
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
  PIN();
  asm volatile("s_barrier" ::: "memory");
  PIN();
  {
    short4v lo;
#pragma unroll
    for (int r = 0; r < NR; ++r) read(smem, smem, 0, r, f[0], lo);
  }
  PIN();

  using T_ = std::true_type;
  using F_ = std::false_type;
  int kt = 0;
  for (; kt < KT - (GK ? 3 : 2); ++kt) kstep(T_{}, T_{}, kt, F_{});
  if constexpr (GK) {
    if (kt < KT - 2) kstep(T_{}, T_{}, kt++, T_{});
  }
  if constexpr (MODE == kTN) {
    if (kt < KT - 1) kstep(F_{}, T_{}, kt++, F_{});
    kstep(F_{}, F_{}, kt, F_{});
  } else {
#pragma unroll 1
    for (; kt < KT; ++kt) kstep(F_{}, T_{}, kt, F_{});
  }
}

// GRAD (kNT only): the epilogue multiplies by act'(pre) read from `pre` [E,C,N], i.e. the product is the gradient with
// respect to the pre-activations of a layer whose activation is ACT; with ACT < 0 it adds `pre` instead (a product
// accumulated onto an existing matrix; `pre` may then be `out` itself, every element being read before it is written
// by the same lane).
// DUAL (kNN with an activation only): the values before the activation are written to `pre_out` as well.
// GK (kTN only): A's k-rows (slots) are gathered through `gather` [E, K] from the matrix A [gather_rows, C] (the token
// matrix, for the first layer's weight gradient when the dispatch buffer was never written).
// FAR (with a gathered A only): see tile_main_loop.
// CUT (not kTN, not FAR): the tiles of the last round may be cut, see cut_tile in ffn_rules.h.
template <int ACT, int MODE, bool GRAD, bool DUAL = false, bool GK = false, bool FAR = false, bool CUT = false>
__global__ __launch_bounds__(kThreads) void grouped_gemm_mfma_kernel(const uint16_t* __restrict__ A,
                                                                     const uint16_t* __restrict__ B,
                                                                     const uint16_t* __restrict__ bias,
                                                                     const int32_t* __restrict__ counts,
                                                                     const int32_t* __restrict__ gather, int gather_rows,
                                                                     int E, int64_t C, int K, int N, int MT, int NT,
                                                                     uint16_t* out,                 // may alias `pre`
                                                                     const int32_t* __restrict__ kfill,
                                                                     const uint16_t* __restrict__ a_tail,
                                                                     const uint16_t* __restrict__ b_tail,
                                                                     const uint16_t* pre,
                                                                     uint16_t* __restrict__ pre_out) {
  __shared__ __attribute__((aligned(1024))) char smem[kRingBytes];

  const int lane = threadIdx.x & 63;
  int e, mt, nt, rows_e;
  TileHalf half;
  if (!find_tile<BM, MODE == kTN, 0, MODE != kTN, CUT>(blockIdx.x, lane, E, C, counts, NT, e, mt, nt, rows_e, half)) return;
  const int64_t rows = rows_e;                                      // already here from the search: no second trip to memory
  const int64_t m0 = (int64_t)mt * BM;
  if (m0 >= rows) return;                                           // cannot happen (mt < mte); keeps every access in the slab
  const int n0 = nt * BN;

  if (CUT && half.col >= 0) {
    const bool tall = rows - m0 > 128;
    if (half.row == 1 && !tall) return;                            // a short tile has no lower half
    Piece p;
    p.m0 = m0 + (half.row == 1 ? 128 : 0);
    p.A = gather ? A : A + (int64_t)e * C * K;
    p.B = B + (int64_t)e * K * N;
    p.n0 = n0 + half.col * 128;
    p.bias = bias ? bias + (int64_t)e * N + p.n0 : nullptr;
    p.gather = gather ? gather + (int64_t)e * C + p.m0 : nullptr;
    p.gather_rows = gather_rows;
    p.rows = (int)(rows - p.m0 < 256 ? rows - p.m0 : 256);
    p.K = K;
    p.N = N;
    p.out = ((int64_t)e * C + p.m0) * N + p.n0;
    if (half.row < 0 && tall) {
      run_piece<256, 128, 3, ACT, MODE, GRAD, DUAL>(smem, p, out, pre, pre_out);
    } else {
      p.rows = p.rows < 128 ? p.rows : 128;
      run_piece<128, 128, 5, ACT, MODE, GRAD, DUAL>(smem, p, out, pre, pre_out);
    }
    return;
  }

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // ---- global sources of this lane's direct-to-LDS loads (32-bit offsets from per-expert scalar bases) -------------
  // Row-major operand with k contiguous (A of kNN/kNT, B of kNT): 1 KB block q*4+wave of the tile = rows
  //   8(q*4+wave) .. +7, lane l writes row +l/8, chunk position l%8.
  // Operand with k as the slow index (B of kNN/kTN, A of kTN): 1 KB block q*4+wave = k-rows 2(q*4+wave), +1, lane l
  //   writes k-row +l/32, chunk position l%32.
  // With `gather` (the slot -> token map [E, C] of the dispatch), A is the token matrix [gather_rows, K] itself and row r
  // of expert e's slab is token gather[e, r]: the dispatch buffer is never written or read.  Unfilled slots (-1) read
  // token 0; their output rows lie past the expert's fill and are never used.
  const char* a_base;
  const char* b_base;
  const char* a_last = nullptr;
  const char* b_last = nullptr;
  int KT = K / BK;
  if (MODE == kTN) {                                                // A [E, K slots, C], B [E, K slots, N]
    a_base = GK ? (const char*)A : (const char*)(A + (int64_t)e * K * C);
    b_base = (const char*)(B + (int64_t)e * K * N);
    int64_t fill = K;
    if (kfill) { const int64_t c = kfill[e]; fill = c < K ? (c > 0 ? c : 0) : K; }
    KT = slot_ksteps(fill);
    a_last = (const char*)(a_tail + (int64_t)e * BK * C);
    b_last = (const char*)(b_tail + (int64_t)e * BK * N);
  } else {
    a_base = gather ? (const char*)A : (const char*)(A + (int64_t)e * C * K);
    b_base = (const char*)(B + (int64_t)e * K * N);
  }
  uint32_t a_voff[8], b_voff[8];
  int a_mask = 0;                                                   // bit q: A block q of this wave holds at least one real row
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int r = (q * 4 + wave) * 8 + (lane >> 3);                 // row of a k-contiguous tile
    const int g = (lane & 7) ^ ((r >> 1) & 7);                      // global chunk that lands at position lane % 8
    const int kr = (q * 4 + wave) * 2 + (lane >> 5);                // k-row of a k-slow tile
    const int c = (lane & 31) ^ (4 * (kr & 3)) ^ (2 * ((kr >> 3) & 1));
    if (MODE == kTN) {
      a_mask |= 1 << q;
      a_voff[q] = (uint32_t)(((int64_t)kr * C + m0 + c * 8) * 2);
    } else {
      if (m0 + (q * 4 + wave) * 8 < rows) a_mask |= 1 << q;
      int64_t row = m0 + r;
      row = row < C ? row : C - 1;                                  // rows past the slab are clamped (never stored)
      if (gather) {
        const int t = gather[(int64_t)e * C + row];
        row = (unsigned)t < (unsigned)gather_rows ? t : 0;
      }
      a_voff[q] = (uint32_t)(FAR ? (row * K + g * 8) >> 3 : (row * K + g * 8) * 2);
    }
    if (MODE == kNT) b_voff[q] = (uint32_t)(((int64_t)(n0 + r) * K + g * 8) * 2);
    else b_voff[q] = (uint32_t)(((int64_t)kr * N + n0 + c * 8) * 2);
  }
  const int64_t a_step = MODE == kTN ? (int64_t)BK * C * 2 : (int64_t)BK * 2;
  const int64_t b_step = MODE == kNT ? (int64_t)BK * 2 : (int64_t)BK * N * 2;

  // ---- LDS read offsets of this lane's MFMA fragments ------------------------------------------------------------
  // direct (k-contiguous tile): row * 128 + ((4 s + kq) ^ (row / 2 % 8)) * 16, one per sub-step s (sub-tile 0; 2048 bytes apart)
  // transposed (k-slow tile):   k-row * 512 + swizzled 16-byte chunk + 8-byte half, one per sub-tile, + (32 s + 4 half) * 512
  const int kg = lane >> 5, kq = lane >> 4;
  auto direct_off = [&](int w, int s) { return (w * 128 + (lane & 15)) * 128 + (((4 * s + kq) ^ ((lane & 15) >> 1)) << 4); };
  auto tr_off = [&](int w, int t) {
    const int kr = (lane & 15) >> 2;                                // k % 4 of the row this lane supplies; k / 8 % 2 = kq % 2
    const int c = w * 16 + t * 2 + ((lane & 3) >> 1);
    return (kq * 8 + kr) * 512 + ((c ^ (4 * kr) ^ (2 * (kq & 1))) << 4) + ((lane & 1) << 3);
  };
  int a_off[8], b_off[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    a_off[i] = MODE == kTN ? tr_off(wm, i) : direct_off(wm, i & 1);
    b_off[i] = kBRing + (MODE == kNT ? direct_off(wn, i & 1) : tr_off(wn, i));
  }
  // 32-row sub-tiles of this wave that hold real rows (the last row tile of an expert is usually ragged)
  const int64_t wave_rows = rows - m0 - wm * 128;
  const int ni = wave_rows >= 128 ? 4 : (wave_rows <= 0 ? 0 : (int)((wave_rows + 31) >> 5));

  f32x4 acc[8][8];
  const uint16_t* bias_w = bias ? bias + (int64_t)e * N + n0 + wn * 128 : nullptr;

  // the number of live sub-tiles is a template argument, so that the loop body of a ragged tile is as branch-free as a
  // full one's (a wave with no rows still loads its share of B and joins the barriers)
#define MOE_TILE_LOOP(NI) tile_main_loop<NI, MODE, false, FAR && MODE == kNN>(smem, a_base, b_base, a_last, b_last, a_voff, b_voff, a_step, b_step, a_off, b_off, kg, kq, a_mask, wave, KT, bias_w, acc)
  if (MODE == kTN && GK) {
    GatherK gk;
    gk.rows = gather + (int64_t)e * K;
    gk.row_bytes = (uint32_t)(C * 2);
    gk.nrows = (uint32_t)gather_rows;
    gk.col = a_voff[0] - (uint32_t)((wave * 2 + kg) * C * 2);       // (m0 + 8 c) * 2: the k-row term taken out again
    gk.tail_step = (uint32_t)(8 * C * 2);
    tile_main_loop<4, MODE, true, FAR>(smem, a_base, b_base, a_last, b_last, a_voff, b_voff, a_step, b_step, a_off, b_off, kg, kq,
                                  a_mask, wave, KT, bias_w, acc, gk);
  } else if (MODE == kTN) {                                         // output rows are a weight dimension: never ragged
    MOE_TILE_LOOP(4);
  } else {
    switch (ni) {
      case 4: MOE_TILE_LOOP(4); break;
      case 3: MOE_TILE_LOOP(3); break;
      case 2: MOE_TILE_LOOP(2); break;
      case 1: MOE_TILE_LOOP(1); break;
      default: MOE_TILE_LOOP(0); break;
    }
  }
#undef MOE_TILE_LOOP

  // ---- epilogue: activation, bf16; transposed through LDS so that global stores are 16 bytes per lane and a
  // wave's store covers 4 rows x 256 contiguous bytes.  After the last barrier of the main loop no direct load is in flight and no
  // wave reads the stages, but for what the last K-step reads ahead and nobody uses, so wave w may use the 32 KB at
  // smem + 32 KB * w as its own [128 rows][16 chunks of 8 columns]; chunk c of row r sits at position c ^ (r % 16), which makes
  // both the 8-byte writes (16 rows per instruction) and the 16-byte row-contiguous reads conflict-free.
  // A DUAL kernel writes the tile twice: first the values before the activation (what a training step keeps for the
  // backward pass), then the activated ones.
  char* wtile = smem + wave * 32768;
  const int64_t out_at = ((int64_t)e * C + m0 + wm * 128) * N + n0 + wn * 128;
  const int64_t live = rows - m0 - wm * 128;                        // rows of this wave's tile that exist
  auto write_tile = [&](auto raw_tag, uint16_t* dst) {
    constexpr bool RAW = decltype(raw_tag)::value;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i >= 2 * ni) break;
      const int r = i * 16 + (lane & 15);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = epilogue_act<(GRAD || RAW) ? -1 : ACT>(acc[i][j][u]);
        u32x2 pk;
        pk.x = pack_bf16x2(v[0], v[1]);
        pk.y = pack_bf16x2(v[2], v[3]);
        *LDS_PTR(u32x2, wtile + r * 256 + (((2 * j + (kq >> 1)) ^ (r & 15)) << 4) + 8 * (kq & 1)) = pk;
      }
    }
    uint16_t* oute = dst + out_at;
    for (int it0 = 0; it0 < 32; it0 += 8) {
      if (it0 * 4 >= ni * 32) break;
      uint4 pv8[8];
      if (GRAD && !RAW) {                                           // this batch's pre-activations, all loads in flight at once
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int r = (it0 + u) * 4 + (lane >> 4);
          const int rr = r < live ? r : 0;                          // rows past the fill: any valid row, result unused
          pv8[u] = *reinterpret_cast<const uint4*>(pre + out_at + (int64_t)rr * N + (((lane & 15) ^ (rr & 15)) << 3));
        }
      }
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const int r = (it0 + u) * 4 + (lane >> 4);
        u32x4 q = *LDS_PTR(u32x4, wtile + r * 256 + ((lane & 15) << 4));
        if (r < live) {
          const int64_t at = (int64_t)r * N + (((lane & 15) ^ (r & 15)) << 3);
          if (GRAD && !RAW) {                                       // times act'(pre), both factors as stored (bf16); or plus `pre`
            float g[8], pv[8];
            Vec16<uint16_t>::unpack(__builtin_bit_cast(uint4, q), g);
            Vec16<uint16_t>::unpack(pv8[u], pv);
#pragma unroll
            for (int v = 0; v < 8; ++v) g[v] = ACT < 0 ? g[v] + pv[v] : g[v] * epilogue_act_grad<ACT>(pv[v]);
            q = __builtin_bit_cast(u32x4, Vec16<uint16_t>::pack(g));
          }
          *reinterpret_cast<u32x4*>(oute + at) = q;
        }
      }
    }
  };
  if (DUAL) write_tile(std::true_type{}, pre_out);
  write_tile(std::false_type{}, out);
}

// dst[e, j, :] = src[e, 64 (KT_e - 1) + j, :] if that slot is below the expert's fill, else 0, for j < 64: the last
// K-step of a kTN product.   src [E, C, W], dst [E, 64, W]; 16-byte pieces, one block per (expert, 4 slots, operand).
struct TailRows {
  const uint4* src;
  uint4* dst;
  const int32_t* gather;        // slot -> row, src is then one matrix
  int64_t gather_rows;
  int cpr;
};
__global__ __launch_bounds__(256) void tail_rows_kernel(const TailRows a, const TailRows b, const int32_t* __restrict__ kfill, int64_t C) {
  const uint4* __restrict__ src = blockIdx.z ? b.src : a.src;
  uint4* __restrict__ dst = blockIdx.z ? b.dst : a.dst;
  const int32_t* __restrict__ gather = blockIdx.z ? b.gather : a.gather;
  const int64_t gather_rows = blockIdx.z ? b.gather_rows : a.gather_rows;
  const int cpr = blockIdx.z ? b.cpr : a.cpr;
  const int e = blockIdx.y;
  int64_t fill = C;
  if (kfill) { const int64_t c = kfill[e]; fill = c < C ? (c > 0 ? c : 0) : C; }
  const int64_t first = (int64_t)(slot_ksteps(fill) - 1) * BK;
  const int j = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int64_t slot = first + j;
  int64_t row = (int64_t)e * C + slot;
  if (gather && slot < fill) {                                      // the slot's row of the gathered matrix
    const int64_t t = gather[row];
    row = t >= 0 && t < gather_rows ? t : 0;
  }
  for (int ch = threadIdx.x & 63; ch < cpr; ch += 64)
    dst[((int64_t)e * BK + j) * cpr + ch] = slot < fill ? src[row * cpr + ch] : make_uint4(0, 0, 0, 0);
}

// `half`: on the half tile; `total`: rows of all experts that exist, at most.
static hipError_t launch_large_nn(const void* A, const void* B, const void* bias, int act, const int32_t* counts,
                                  int64_t E, int64_t C, int64_t K, int64_t N, void* out, hipStream_t s, bool half, int64_t total,
                                  int64_t rows_hint, const int32_t* gather, int64_t gather_rows, void* pre_out) {
  const int64_t bm = half ? BM / 2 : BM;
  const int MT = (int)ceil_div(C, bm), NT = (int)(N / BN);
  const bool cut = !half && !far_rows(gather_rows, K) && cuts_last_round(E, C, mean_or(rows_hint, C), counts, NT);
  const int64_t blocks = tile_grid(NT, live_row_tiles(E, C, total, bm), true, cut);
  if (blocks >= kMaxBlocks) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(kThreads);
#define MOE_LAUNCH_GEMM_AT(ACT, DUAL, FAR, CUT)                                                                       \
  grouped_gemm_mfma_kernel<ACT, kNN, false, DUAL, false, FAR, CUT><<<grid, block, 0, s>>>(                                 \
      (const uint16_t*)A, (const uint16_t*)B, (const uint16_t*)bias, counts, gather, (int)gather_rows, (int)E, C,     \
      (int)K, (int)N, MT, NT, (uint16_t*)out, nullptr, nullptr, nullptr, nullptr,                                       \
      (uint16_t*)pre_out)
#define MOE_LAUNCH_GEMM(ACT, DUAL)                                                                                    \
  do {                                                                                                                \
    if (half)                                                                                                         \
      grouped_gemm_half_kernel<ACT><<<grid, block, 0, s>>>((const uint16_t*)A, (const uint16_t*)B, (const uint16_t*)bias, \
                                                           counts, gather, (int)gather_rows, (int)E, C, (int)K, (int)N, MT, NT, (uint16_t*)out); \
    else if (far_rows(gather_rows, K)) MOE_LAUNCH_GEMM_AT(ACT, DUAL, true, false);                                     \
    else if (cut) MOE_LAUNCH_GEMM_AT(ACT, DUAL, false, true);                                                         \
    else MOE_LAUNCH_GEMM_AT(ACT, DUAL, false, false);                                                                 \
  } while (0)
  if (pre_out && act >= 0) {
    switch (act) {
      case MOE_ACT_RELU: MOE_LAUNCH_GEMM(MOE_ACT_RELU, true); break;
      case MOE_ACT_GELU: MOE_LAUNCH_GEMM(MOE_ACT_GELU, true); break;
      default: MOE_LAUNCH_GEMM(MOE_ACT_SILU, true); break;
    }
  } else {
    switch (act) {
      case MOE_ACT_RELU: MOE_LAUNCH_GEMM(MOE_ACT_RELU, false); break;
      case MOE_ACT_GELU: MOE_LAUNCH_GEMM(MOE_ACT_GELU, false); break;
      case MOE_ACT_SILU: MOE_LAUNCH_GEMM(MOE_ACT_SILU, false); break;
      default: MOE_LAUNCH_GEMM(-1, false); break;
    }
  }
#undef MOE_LAUNCH_GEMM
#undef MOE_LAUNCH_GEMM_AT
  return hipGetLastError();
}

// out[e] = A[e] (rows_e x K) * Bt[e]^T, Bt [E, N, K]; with `pre` [E, C, N] the result is multiplied by act'(pre), or,
// with act < 0, has `pre` added (pre == out accumulates in place).
static hipError_t launch_large_nt(const void* A, const void* Bt, const int32_t* counts, int64_t E, int64_t C,
                                  int64_t K, int64_t N, void* out, const void* pre, int act, hipStream_t s, int64_t total, int64_t rows_hint) {
  const int MT = (int)ceil_div(C, BM), NT = (int)(N / BN);
  const bool cut = cuts_last_round(E, C, mean_or(rows_hint, C), counts, NT);
  const int64_t blocks = tile_grid(NT, live_row_tiles(E, C, total, BM), true, cut);
  if (blocks >= kMaxBlocks) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(kThreads);
#define MOE_LAUNCH_GEMM_AT(ACT, GRAD, CUT)                                                                            \
  grouped_gemm_mfma_kernel<ACT, kNT, GRAD, false, false, false, CUT><<<grid, block, 0, s>>>(                          \
      (const uint16_t*)A, (const uint16_t*)Bt, nullptr, counts, nullptr, 0, (int)E, C, (int)K, (int)N, MT, NT,        \
      (uint16_t*)out, nullptr, nullptr, nullptr, (const uint16_t*)pre, nullptr)
#define MOE_LAUNCH_GEMM(ACT, GRAD)                                                                                    \
  do {                                                                                                                \
    if (cut) MOE_LAUNCH_GEMM_AT(ACT, GRAD, true);                                                                     \
    else MOE_LAUNCH_GEMM_AT(ACT, GRAD, false);                                                                        \
  } while (0)
  if (!pre) MOE_LAUNCH_GEMM(-1, false);
  else if (act < 0) MOE_LAUNCH_GEMM(-1, true);                      // out = product + pre
  else switch (act) {
    case MOE_ACT_RELU: MOE_LAUNCH_GEMM(MOE_ACT_RELU, true); break;
    case MOE_ACT_GELU: MOE_LAUNCH_GEMM(MOE_ACT_GELU, true); break;
    default: MOE_LAUNCH_GEMM(MOE_ACT_SILU, true); break;
  }
#undef MOE_LAUNCH_GEMM
#undef MOE_LAUNCH_GEMM_AT
  return hipGetLastError();
}

// out[e] (R x N) = At[e]^T * B[e] over the first min(kfill[e], C) of the C slots; At [E, C, R], B [E, C, N], R and N
// multiples of 256.  a_tail [E, 64, R] and b_tail [E, 64, N] are scratch for the zero-padded last K-step.
// With `gather` [E, C] (slot -> row, as the dispatch builds it) At is one matrix [gather_rows, R] and slot c of expert e
// is its row gather[e, c].
static hipError_t launch_large_tn(const void* At, const void* B, const int32_t* kfill, int64_t E, int64_t C, int64_t R,
                                  int64_t N, void* a_tail, void* b_tail, void* out, hipStream_t s, const int32_t* gather,
                                  int64_t gather_rows) {
  const TailRows ta = {(const uint4*)At, (uint4*)a_tail, gather, gather_rows, (int)(R / 8)}, tb = {(const uint4*)B, (uint4*)b_tail, nullptr, 0, (int)(N / 8)};
  tail_rows_kernel<<<dim3(BK / 4, (unsigned)E, 2), dim3(256), 0, s>>>(ta, tb, kfill, C);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const int MT = (int)(R / BM), NT = (int)(N / BN);
  const int64_t blocks = tile_grid(NT, E * MT);
  if (blocks >= kMaxBlocks) return hipErrorInvalidValue;
  const dim3 grid((unsigned)blocks), block(kThreads);
#define MOE_LAUNCH_GATHERED(FAR)                                                                                        \
  grouped_gemm_mfma_kernel<-1, kTN, false, false, true, FAR><<<grid, block, 0, s>>>(                                    \
      (const uint16_t*)At, (const uint16_t*)B, nullptr, nullptr, gather, (int)gather_rows, (int)E, R, (int)C, (int)N, MT, NT, \
      (uint16_t*)out, kfill, (const uint16_t*)a_tail, (const uint16_t*)b_tail, nullptr, nullptr)
  if (gather && far_rows(gather_rows, R)) MOE_LAUNCH_GATHERED(true);
  else if (gather) MOE_LAUNCH_GATHERED(false);
#undef MOE_LAUNCH_GATHERED
  else
    grouped_gemm_mfma_kernel<-1, kTN, false><<<grid, block, 0, s>>>(
        (const uint16_t*)At, (const uint16_t*)B, nullptr, nullptr, nullptr, 0, (int)E, R, (int)C, (int)N, MT, NT,
        (uint16_t*)out, kfill, (const uint16_t*)a_tail, (const uint16_t*)b_tail, nullptr, nullptr);
  return hipGetLastError();
}

bool grouped_gemm_gathers_on_large_tile(int64_t E, int64_t C, int64_t K, int64_t N, int64_t gather_rows) {
  return large_tile_supports(E, C, K, N, gather_rows) && !far_rows(gather_rows, K);
}

// Rows that exist in all, at most.  Only a caller that counts has a hint that is also a promise.
static int64_t total_rows(const int32_t* counts, int64_t E, int64_t C, int64_t rows_hint) {
  return E * (counts && rows_hint > 0 && rows_hint < C ? rows_hint : C);
}

hipError_t launch_grouped_gemm(const void* A, const void* B, const void* bias, int act, int dtype, const int32_t* counts,
                               int64_t E, int64_t C, int64_t K, int64_t N, void* out, hipStream_t s, int64_t rows_hint,
                               void* pre_out, const int32_t* gather, int64_t gather_rows) {
  if (act < 0) pre_out = nullptr;                                   // nothing to tell apart
  const Tile tile = dtype == MOE_BF16 ? tile_of(kNN, E, C, K, N, rows_hint, gather ? gather_rows : 0, pre_out != nullptr) : Tile::k64;
  const int64_t total = total_rows(counts, E, C, rows_hint);
  if (tile == Tile::k256 || tile == Tile::kHalf)
    return launch_large_nn(A, B, bias, act, counts, E, C, K, N, out, s, tile == Tile::kHalf, total, rows_hint, gather, gather_rows, pre_out);
  if (dtype == MOE_BF16 && act > MOE_ACT_RELU && !large_tile_supports(E, C, K, N, 0)) act += kFullAct;
  const TileArgs p = {A, B, bias, counts, gather, gather_rows, C, K, (int)N, (int)E, 0, 0, 0, out, nullptr, nullptr, pre_out, act, 0};
  return launch_small<kNN>(dtype, tile, p, total, s);
}

// out[e] = A[e] (rows_e x K) * Bt[e]^T, Bt [E, N, K]; with `pre` [E, C, N] the result is multiplied by act'(pre), or,
// with act < 0, has `pre` added (pre == out accumulates in place).
hipError_t launch_grouped_gemm_nt(const void* A, const void* Bt, int dtype, const int32_t* counts, int64_t E, int64_t C,
                                  int64_t K, int64_t N, void* out, const void* pre, int act, hipStream_t s, int64_t rows_hint) {
  const Tile tile = dtype == MOE_BF16 ? tile_of(kNT, E, C, K, N, rows_hint, 0, false) : Tile::k64;
  const int64_t total = total_rows(counts, E, C, rows_hint);
  if (tile == Tile::k256) return launch_large_nt(A, Bt, counts, E, C, K, N, out, pre, act, s, total, rows_hint);
  if (dtype == MOE_BF16 && act > MOE_ACT_RELU && !large_tile_supports_backward(E, C, K, N)) act += kFullAct;
  const TileArgs p = {A, Bt, nullptr, counts, nullptr, 0, C, K, (int)N, (int)E, 0, 0, 0, out, nullptr, pre, nullptr, pre ? act : -1, 0};
  return launch_small<kNT>(dtype, tile, p, total, s);
}

size_t grouped_gemm_tn_tail_bytes(int64_t E, int64_t W) { return (size_t)E * BK * W * 2; }

// out[e] (R x N) = At[e]^T * B[e] over the first min(kfill[e], C) of the C slots; At [E, C, R], B [E, C, N].  a_tail and
// b_tail: scratch of grouped_gemm_tn_tail_bytes(E, R) and (E, N).  With `gather` [E, C] At is one matrix [gather_rows, R] and
// slot c of expert e is its row gather[e, c].
hipError_t launch_grouped_gemm_tn(const void* At, const void* B, int dtype, const int32_t* kfill, int64_t E, int64_t C, int64_t R,
                                  int64_t N, void* a_tail, void* b_tail, void* out, hipStream_t s, int64_t rows_hint,
                                  const int32_t* gather, int64_t gather_rows) {
  const Tile tile = dtype == MOE_BF16 ? tile_of(kTN, E, R, C, N, rows_hint, gather_rows, false) : Tile::k64;
  if (tile == Tile::k256) return launch_large_tn(At, B, kfill, E, C, R, N, a_tail, b_tail, out, s, gather, gather_rows);
  const TileArgs p = {At, B, nullptr, nullptr, gather, gather_rows, R, C, (int)N, (int)E, 0, 0, 0, out, kfill, nullptr, nullptr, -1, 0};
  return launch_small<kTN>(dtype, tile, p, E * R, s);
}

// The reduction of a kTN product with one small result, cut into slices whose sums leave as fp32: see common.h.
template <typename ET, int BM, int BN, int WR, int WC>
static hipError_t launch_slices(TileArgs p, hipStream_t s) {
  p.MT = (int)ceil_div(p.C, BM);
  p.NT = (int)ceil_div(p.N, BN);
  const int64_t blocks = tile_grid(p.NT, (int64_t)p.E * p.MT);
  if (blocks >= kMaxBlocks) return hipErrorInvalidValue;
  grouped_gemm_tile_kernel<ET, kTN, BM, BN, WR, WC, 2, false, true><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(p);
  return hipGetLastError();
}

// Columns of a slice's tile: no more than the results have, as far as a matrix instruction is not narrower still.  (fp32, 65536
// tokens, M = 2048, dWg of 8 experts: 163 us with 64, 106 with 32.)
static int slices_width(int dtype, int64_t N) { return N <= 32 ? 32 : (N <= 64 || dtype == MOE_F32 ? 64 : 128); }
static int slices_height(int dtype, int64_t N) { return dtype == MOE_F32 && N > 32 ? 64 : 128; }

// Enough slices for about four blocks per compute unit, but no more than 64 (their sums are written and read again) and no more
// than one to 256 k; a slice is a whole number of K-steps.
GemmSlices gemm_slices(int dtype, int64_t K, int64_t R, int64_t N) {
  const int64_t tiles = ceil_div(R, slices_height(dtype, N)) * ceil_div(N, slices_width(dtype, N));
  int64_t n = ceil_div(1024, tiles);
  n = n < 64 ? n : 64;
  n = n < ceil_div(K, 256) ? n : ceil_div(K, 256);
  GemmSlices g;
  g.length = ceil_div(ceil_div(K, n), 64) * 64;
  g.count = ceil_div(K, g.length);
  return g;
}

hipError_t launch_gemm_tn_slices(const void* At, const void* B, int dtype, int64_t K, int64_t R, int64_t N, float* out, hipStream_t s) {
  const GemmSlices g = gemm_slices(dtype, K, R, N);
  TileArgs p = {At, B, nullptr, nullptr, nullptr, 0, R, g.length, (int)N, (int)g.count, 0, 0, 0, out, nullptr, nullptr, nullptr, -1, K};
  if (dtype == MOE_F32) return N <= 32 ? launch_slices<float, 128, 32, 4, 1>(p, s) : launch_slices<float, 64, 64, 2, 2>(p, s);
  switch (slices_width(dtype, N)) {
    case 32: return launch_slices<uint16_t, 128, 32, 4, 1>(p, s);
    case 64: return launch_slices<uint16_t, 128, 64, 2, 2>(p, s);
    default: return launch_slices<uint16_t, 128, 128, 2, 2>(p, s);
  }
}

}  // namespace moe
