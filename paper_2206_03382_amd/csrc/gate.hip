// Gating function and capacity-limited slot assignment (arXiv 2206.03382 Sec. 2.1, Eq. 1; Appendix B names the
// location scan).  The kernels of the gate:
//   gate_logits_kernel : logits = x * Wg + bias on the fp64 matrix cores (order-independent after rounding to fp32)
//                        (gate_logits_wide_kernel: wide gates and many tokens)
//   gate_topk_kernel   : per token softmax + k rounds of (value, index) argmax in a sub-wave group; per-block,
//                        per-rank, per-expert arrival counters
//   gate_scan_kernel   : per expert, exclusive scan of the counters in arrival order (rank, block); totals;
//                        marks unfilled slots of slot_src with -1
//   gate_assign_kernel : per token and rank, position inside its block + scanned offset -> loc, slot_src
//                        (gate_slots_kernel: scan and assignment at once where the counters are few)
// No order-dependent atomics: every integer output is a pure function of the logits.
// Further down: the dynamic capacity factor and slot sources for a capacity chosen after routing (Sec. 4.1), the cosine
// router (Appendix), and the token order of batch prioritized routing (Sec. 3.2 / Appendix ablation).
#include "common.h"
#include "gate_rules.h"

namespace moe {

typedef __attribute__((ext_vector_type(4))) double f64x4;

// ---------------------------------------------------------------------------------------------------------------
// logits[t,e] = sum_m x[t,m] Wg[m,e] + bias[e], fp64 accumulate (v_mfma_f64_16x16x4_f64), one rounding to fp32.
// A wave owns 16 tokens and NT tiles of 16 experts.  Operand layout of the instruction: A lane l holds
// (row l%16, k l/16), B lane l holds (k l/16, col l%16), D lane l register v holds (row 4v + l/16, col l%16).
// A lane keeps 8 consecutive x values (k = kq*8 .. kq*8+7 of a 32-wide chunk); MFMA step s uses k = kq*8+s for
// both operands, so the chunk's 32 k-values are covered exactly once.
// ---------------------------------------------------------------------------------------------------------------
// N consecutive values of a row as floats, kept raw while in flight
template <typename XT, int N> struct RawN {
  uint32_t w[N * (int)sizeof(XT) / 4];
  __device__ __forceinline__ void load_vec(const XT* p) {                        // aligned to N * sizeof(XT) = 8, 16 or 32 bytes
    if constexpr (N * sizeof(XT) == 8) {
      const uint2 v = *reinterpret_cast<const uint2*>(p);
      w[0] = v.x; w[1] = v.y;
    } else {
#pragma unroll
      for (int i = 0; i < N * (int)sizeof(XT) / 16; ++i) {
        const uint4 v = reinterpret_cast<const uint4*>(p)[i];
        w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
      }
    }
  }
  __device__ __forceinline__ void keep_if(bool on) {
#pragma unroll
    for (int i = 0; i < N * (int)sizeof(XT) / 4; ++i) w[i] = on ? w[i] : 0u;
  }
  __device__ __forceinline__ float get(int i) const {
    if constexpr (sizeof(XT) == 4) return __uint_as_float(w[i]);
    else return __uint_as_float((i & 1) ? w[i >> 1] & 0xffff0000u : w[i >> 1] << 16);
  }
  __device__ __forceinline__ void set(int i, XT v) {
    if constexpr (sizeof(XT) == 4) w[i] = __float_as_uint(v);
    else w[i >> 1] = (i & 1) ? (w[i >> 1] & 0xffffu) | ((uint32_t)v << 16) : (uint32_t)v;
  }
};

// Gates of up to 64 experts, few tokens, and what wide gates leave over: a wave owns TW tiles of 16 tokens x NT tiles of 16 experts over
// one of KS parts of the reduction, a block the KS parts of its tiles, whose sums are added in part order through LDS.  Both
// operands come straight from global memory, two passes of 32 k ahead in registers: x once in 16-byte pieces, Wg (which every
// wave reads, so from the caches) element by element in the layout the instruction wants.  No barrier and no LDS in the
// loop, so waves drift apart and cover each other's loads.  Binds: the fp64 matrix pipe (16 columns are computed whatever E
// is) and beside it the element loads of Wg; for few tokens the chain of M / (32 KS) passes, hence KS = 16 there.
// Measured against four waves on fp64 weights staged through LDS, in a captured graph with its launch: 512 tokens, M = 1024,
// 64 experts, fp32 53 -> 17 us; 64 tokens, M = 4096, 64 experts 180 -> 20; 16384 tokens, M = 2048, 8 experts 41 -> 35.
template <typename XT, int NT, int KS, int TW>
__device__ __forceinline__ void logits_of_tiles(const XT* __restrict__ x, const XT* __restrict__ Wg, const float* __restrict__ bias, int64_t T, int M,
                                                int E, int64_t t0, int e0, float* __restrict__ logits) {
  constexpr int PF = 2;
  __shared__ double red[KS - 1][TW * NT][4][64];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, kq = lane >> 4;
  const int passes = (M + 31) / 32, per = (passes + KS - 1) / KS;
  const int p0 = wave * per, p1 = p0 + per < passes ? p0 + per : passes;   // this wave's passes (possibly none)
  const XT* xrow[TW];
#pragma unroll
  for (int w = 0; w < TW; ++w) {
    const int64_t t = t0 + w * 16 + r;
    xrow[w] = x + (t < T ? t : T - 1) * (int64_t)M;
  }
  int ecol[NT];                                                     // columns past the last repeat it and are never stored
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) ecol[nt] = e0 + nt * 16 + r < E ? e0 + nt * 16 + r : E - 1;
  RawN<XT, 8> xr[PF][TW];
  XT wr[PF][NT][8];
  auto fetch = [&](int slot, int p) __attribute__((always_inline)) { // k past the row's end: the row's start is read and zeroed
    const int k = p * 32 + kq * 8;
    const bool live = k < M;
#pragma unroll
    for (int w = 0; w < TW; ++w) {
      xr[slot][w].load_vec(xrow[w] + (live ? k : 0));
      xr[slot][w].keep_if(live);
    }
    const XT* wp = Wg + (int64_t)(live ? k : 0) * E;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const XT v = wp[(int64_t)u * E + ecol[nt]];
        wr[slot][nt][u] = live ? v : (XT)0;
      }
  };
  f64x4 acc[TW][NT];
#pragma unroll
  for (int w = 0; w < TW; ++w)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[w][nt] = f64x4{0.0, 0.0, 0.0, 0.0};
  auto compute = [&](int slot) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        const double b = (double)load_as_f32<XT>(&wr[slot][nt][u]);
#pragma unroll
        for (int w = 0; w < TW; ++w) acc[w][nt] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)xr[slot][w].get(u), b, acc[w][nt], 0, 0, 0);
      }
  };
#pragma unroll
  for (int q = 0; q < PF; ++q)
    if (p0 + q < p1) fetch(q, p0 + q);
  for (int p = p0; p < p1; p += PF) {
#pragma unroll
    for (int q = 0; q < PF; ++q) {
      if (p + q >= p1) break;
      compute(q);
      if (p + q + PF < p1) fetch(q, p + q + PF);
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int w = 0; w < TW; ++w)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave - 1][w * NT + nt][v][lane] = acc[w][nt][v];
  }
  __syncthreads();
  if (wave > 0) return;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int e = e0 + nt * 16 + r;
    const double be = bias && e < E ? (double)bias[e] : 0.0;
#pragma unroll
    for (int w = 0; w < TW; ++w) {
#pragma unroll
      for (int q = 1; q < KS; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc[w][nt][v] += red[q - 1][w * NT + nt][v][lane];
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t t = t0 + w * 16 + 4 * v + kq;
        if (t < T && e < E) logits[t * E + e] = (float)(acc[w][nt][v] + be);
      }
    }
  }
}

template <typename XT, int NT, int KS, int TW>
__global__ __launch_bounds__(64 * KS) void gate_logits_kernel(const XT* __restrict__ x, const XT* __restrict__ Wg,
                                                              const float* __restrict__ bias, int64_t T, int M, int E,
                                                              int e_base, float* __restrict__ logits) {
  logits_of_tiles<XT, NT, KS, TW>(x, Wg, bias, T, M, E, (int64_t)blockIdx.x * (16 * TW), e_base + blockIdx.y * (16 * NT), logits);
}

// Wide gates of many tokens (the cosine router's projection; the rule: gate_rules.h): a block's 2 x 2 waves own 32 tokens x 64 experts, a wave
// 16 x 32 as two accumulator tiles.  Both operands go through LDS in 32 bits, 32 k at a time (the next 32 k are fetched to
// registers meanwhile): fp32 values are widened on the way out; of bf16 values, widened on the way in, LDS holds the upper half of the fp64.  Per 32 k a
// wave issues 16 matrix instructions of 64 cycles against 18 LDS reads, which hide behind them, and 13 KB of LDS let eight blocks share a unit and cover each
// other's staging.  What binds is the fp64 matrix pipe and beside it the conversions.  Blocks are small because the count of blocks per unit is what
// divides unevenly; all expert blocks go in one launch.  Replaced blocks of 128 experts, seven to a unit, both operands in fp32: 25088 tokens, M = 768, 256
// columns 203 -> 186 us (53 TFLOP/s; the fp64 matrix pipe alone sustains 67), of which the conversions 3 us by the profiler; fp32, 65536 tokens, M = 2048, 128
// experts 632 -> 598; over 300 gates of 104 to 512 experts between 0.87 and 1.01 of their time from M = 256 on, with M = 64 up to 1.03 (201650 tokens, 104 experts 68.6 and 70.7).  (Those replaced four waves of 16 tokens x 128 experts on fp64 weights in LDS, 275 us.)
// LDS rows: 36 values per token (16 rows x 4 groups of a ds_read_b128 spread over all banks), 66 per k of the weights (the
// four k of an operand read lie 16 banks apart).
constexpr int kWideTokens = 32, kWideExperts = 64, kWideK = 32, kWideLdx = 36, kWideLdw = 66;

// What LDS holds of an operand, in 32 bits: of a bf16 value widened to fp64 the upper half (the lower one is zero), else the fp32 value.
template <typename XT> __device__ __forceinline__ float wide_store(float v) {
  if constexpr (sizeof(XT) == 2) return __uint_as_float((uint32_t)(__builtin_bit_cast(uint64_t, (double)v) >> 32));
  else return v;
}
template <typename XT> __device__ __forceinline__ double wide_load(float v) {
  if constexpr (sizeof(XT) == 2) return __builtin_bit_cast(double, (uint64_t)__float_as_uint(v) << 32);
  else return (double)v;
}

// E a multiple of 8 and Wg 16-byte aligned.
template <typename XT>
__global__ __launch_bounds__(256, 8) void gate_logits_wide_kernel(const XT* __restrict__ x, const XT* __restrict__ Wg,
                                                               const float* __restrict__ bias, int64_t T, int M, int E,
                                                               int expert_blocks, float* __restrict__ logits) {
  __shared__ __attribute__((aligned(16))) float xs[kWideTokens * kWideLdx];
  __shared__ __attribute__((aligned(16))) float ws[kWideK * kWideLdw];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4, wt = wave >> 1, we = wave & 1;
  const int64_t t0 = (int64_t)(blockIdx.x / expert_blocks) * kWideTokens;       // the blocks that share tokens run together
  const int e0 = (int)(blockIdx.x % expert_blocks) * kWideExperts;

  // staging: thread i brings 4 values of token i / 8 and 8 of k row i / 8
  const int srow = threadIdx.x >> 3, sp = threadIdx.x & 7;
  const int64_t st = t0 + srow < T ? t0 + srow : T - 1;
  const XT* xsrc = x + st * (int64_t)M + sp * 4;
  const int we0 = e0 + sp * 8;                                      // first expert of this thread's 8
  RawN<XT, 4> xr;
  RawN<XT, 8> wr;
  auto fetch = [&](int k0) __attribute__((always_inline)) {          // M is a multiple of 8: four values are all inside or all outside
    const bool live = k0 + sp * 4 < M;
    xr.load_vec(live ? xsrc + k0 : xsrc - sp * 4);
    xr.keep_if(live);
    const bool wlive = k0 + srow < M;
    const XT* row = Wg + (int64_t)(wlive ? k0 + srow : 0) * E;
    wr.load_vec(row + (we0 < E ? we0 : 0));
    wr.keep_if(wlive && we0 < E);
  };
  f64x4 acc[2];
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) acc[nt] = f64x4{0.0, 0.0, 0.0, 0.0};
  fetch(0);
  for (int k0 = 0; k0 < M; k0 += kWideK) {
    __syncthreads();                                                // the previous chunk has been read
    *reinterpret_cast<float4*>(&xs[srow * kWideLdx + sp * 4]) = make_float4(wide_store<XT>(xr.get(0)), wide_store<XT>(xr.get(1)), wide_store<XT>(xr.get(2)), wide_store<XT>(xr.get(3)));
#pragma unroll
    for (int u = 0; u < 8; u += 2) *reinterpret_cast<float2*>(&ws[srow * kWideLdw + sp * 8 + u]) = make_float2(wide_store<XT>(wr.get(u)), wide_store<XT>(wr.get(u + 1)));
    __syncthreads();
    if (k0 + kWideK < M) fetch(k0 + kWideK);
    const float* xa = &xs[(wt * 16 + r) * kWideLdx + kq * 8];
    const float4 a0 = *reinterpret_cast<const float4*>(xa), a1 = *reinterpret_cast<const float4*>(xa + 4);
    const float av[8] = {a0.x, a0.y, a0.z, a0.w, a1.x, a1.y, a1.z, a1.w};
    const float* wb = &ws[kq * 8 * kWideLdw + we * 32 + r];
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
        acc[nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(wide_load<XT>(av[s]), wide_load<XT>(wb[s * kWideLdw + nt * 16]), acc[nt], 0, 0, 0);
  }
#pragma unroll
  for (int nt = 0; nt < 2; ++nt) {
    const int e = e0 + we * 32 + nt * 16 + r;
    if (e >= E) continue;
    const double be = bias ? (double)bias[e] : 0.0;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t t = t0 + wt * 16 + 4 * v + kq;
      if (t < T) logits[t * E + e] = (float)(acc[nt][v] + be);
    }
  }
}

// Experts e_base .. end - 1 (end: E, or a whole number of tiles on)
template <typename XT, int NT, int KS, int TW>
static void launch_gate_logits_one(const XT* x, const XT* Wg, const float* bias, int64_t T, int64_t M, int64_t E, int64_t e_base,
                                   int64_t end, float* logits, hipStream_t s) {
  const dim3 grid((unsigned)ceil_div(T, 16 * TW), (unsigned)ceil_div(end - e_base, 16 * NT));
  gate_logits_kernel<XT, NT, KS, TW><<<grid, dim3(64 * KS), 0, s>>>(x, Wg, bias, T, (int)M, (int)E, (int)e_base, logits);
}

// Tokens to a launch: a grid dimension holds fewer than 2^32 threads, 256 to every 16 tokens or, for wide gates, to every 32
// tokens and 64 experts.
static int64_t gate_logits_tokens_per_launch(int64_t E) {
  const int64_t n = ((int64_t)1 << 27) / (E > 64 ? ceil_div(E, kWideExperts) : 1) / kWideTokens * kWideTokens;
  return n > kWideTokens ? n : kWideTokens;
}

template <typename XT>
static hipError_t launch_gate_logits_t(const XT* x, const XT* Wg, const float* bias, int64_t T, int64_t M, int64_t E,
                                       float* logits, hipStream_t s) {
  const int64_t most = gate_logits_tokens_per_launch(E);
  for (; T > most; T -= most, x += most * M, logits += most * E) {
    const hipError_t err = launch_gate_logits_t<XT>(x, Wg, bias, most, M, E, logits, s);
    if (err != hipSuccess) return err;
  }
  // few tiles of 16 tokens x 16 experts: one to a block of 16 waves, whatever E is.  At 512 tiles as fast as four waves with
  // all of a gate's experts, below up to three times as fast (64 tokens, M = 4096, 64 experts: 20 us against 67).
  if (gate_logits_few_tiles(T, E)) {
    launch_gate_logits_one<XT, 1, 16, 1>(x, Wg, bias, T, M, E, 0, E, logits, s);
    return hipGetLastError();
  }
  // Experts below `wide` go to the wide kernel, the others to the narrow one, 64 at a time and then what is left.
  const bool vecw = E % 8 == 0 && ((uintptr_t)Wg & 15) == 0;
  const int64_t wide = gate_logits_wide_experts(T, E, vecw);
  if (wide > 0) {
    const int64_t expert_blocks = ceil_div(wide, kWideExperts), blocks = ceil_div(T, kWideTokens) * expert_blocks;
    gate_logits_wide_kernel<XT><<<dim3((unsigned)blocks), dim3(256), 0, s>>>(x, Wg, bias, T, (int)M, (int)E, (int)expert_blocks, logits);
  }
  // The narrow kernel's waves: two token tiles halve the reads of Wg and eight parts of the reduction shorten its chain, each where
  // enough blocks are left (bf16, M = 4096: 12000 tokens, 32 experts, eight parts and four 74 and 79 us; 16384 with two token
  // tiles 86, with one 95; 16384, 64 experts, two and one 165 and 183; 8200 157 and 135).
  int64_t e = wide;
  if (E - e > 32) {
    const int64_t end = E - e <= 64 ? E : E - (E - e) % 64;
    if (T >= 16384) launch_gate_logits_one<XT, 4, 4, 2>(x, Wg, bias, T, M, E, e, end, logits, s);
    else launch_gate_logits_one<XT, 4, 4, 1>(x, Wg, bias, T, M, E, e, end, logits, s);
    e = end;
  }
  if (E - e > 32) {
    if (T >= 16384) launch_gate_logits_one<XT, 4, 4, 2>(x, Wg, bias, T, M, E, e, E, logits, s);
    else launch_gate_logits_one<XT, 4, 4, 1>(x, Wg, bias, T, M, E, e, E, logits, s);
  } else if (E - e > 16) {
    if (T >= 16384) launch_gate_logits_one<XT, 2, 8, 2>(x, Wg, bias, T, M, E, e, E, logits, s);
    else launch_gate_logits_one<XT, 2, 8, 1>(x, Wg, bias, T, M, E, e, E, logits, s);
  } else if (E > e) {
    if (T >= 32768) launch_gate_logits_one<XT, 1, 4, 2>(x, Wg, bias, T, M, E, e, E, logits, s);
    else launch_gate_logits_one<XT, 1, 8, 1>(x, Wg, bias, T, M, E, e, E, logits, s);
  }
  return hipGetLastError();
}

hipError_t launch_gate_logits(const void* x, const void* Wg, const float* bias, int dtype, int64_t T, int64_t M,
                              int64_t E, float* logits, hipStream_t s) {
  if (dtype == MOE_F32) return launch_gate_logits_t<float>((const float*)x, (const float*)Wg, bias, T, M, E, logits, s);
  return launch_gate_logits_t<uint16_t>((const uint16_t*)x, (const uint16_t*)Wg, bias, T, M, E, logits, s);
}

// ---------------------------------------------------------------------------------------------------------------
// softmax + top-k.  A group of G lanes (power of two, <= 64) owns one token; lane gl holds experts gl, gl+G, ...
// (V per lane).  Selection is k rounds of argmax on (value, index): larger value wins, equal values -> lower
// index, so the result is unique and independent of the reduction tree.
// ---------------------------------------------------------------------------------------------------------------
// Value of the partner lane in one step of a reduction over a group of lanes.  Steps 1 and 2 swap within quads, steps 4
// and 8 read the mirrored lane of the other half of 8 / 16 lanes (data-parallel primitives, no LDS traffic); the mirror
// is as good as an xor partner wherever the lanes of each half already agree, which holds in a reduction whose steps run
// in ascending order.  Steps 16 and 32 go through the cross-lane permute.
template <int OFF> __device__ __forceinline__ int group_partner(int v) {
  if constexpr (OFF == 1) return __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xf, 0xf, false);        // quad_perm [1,0,3,2]
  else if constexpr (OFF == 2) return __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xf, 0xf, false);   // quad_perm [2,3,0,1]
  else if constexpr (OFF == 4) return __builtin_amdgcn_update_dpp(0, v, 0x141, 0xf, 0xf, false);  // row_half_mirror
  else if constexpr (OFF == 8) return __builtin_amdgcn_update_dpp(0, v, 0x140, 0xf, 0xf, false);  // row_mirror
  else return __shfl_xor(v, OFF, 64);
}
template <int OFF> __device__ __forceinline__ float group_partner(float v) {
  return __int_as_float(group_partner<OFF>(__float_as_int(v)));
}

template <int G> __device__ __forceinline__ float group_max(float v) {
  if constexpr (G > 1) v = fmaxf(v, group_partner<1>(v));
  if constexpr (G > 2) v = fmaxf(v, group_partner<2>(v));
  if constexpr (G > 4) v = fmaxf(v, group_partner<4>(v));
  if constexpr (G > 8) v = fmaxf(v, group_partner<8>(v));
  if constexpr (G > 16) v = fmaxf(v, group_partner<16>(v));
  if constexpr (G > 32) v = fmaxf(v, group_partner<32>(v));
  return v;
}
template <int G> __device__ __forceinline__ float group_sum(float v) {
  if constexpr (G > 1) v += group_partner<1>(v);
  if constexpr (G > 2) v += group_partner<2>(v);
  if constexpr (G > 4) v += group_partner<4>(v);
  if constexpr (G > 8) v += group_partner<8>(v);
  if constexpr (G > 16) v += group_partner<16>(v);
  if constexpr (G > 32) v += group_partner<32>(v);
  return v;
}
template <int OFF> __device__ __forceinline__ void argmax_step(float& bv, int& be) {
  const float ov = group_partner<OFF>(bv);
  const int oe = group_partner<OFF>(be);
  if (ov > bv || (ov == bv && oe < be)) { bv = ov; be = oe; }
}
template <int G> __device__ __forceinline__ void group_argmax(float& bv, int& be) {
  if constexpr (G > 1) argmax_step<1>(bv, be);
  if constexpr (G > 2) argmax_step<2>(bv, be);
  if constexpr (G > 4) argmax_step<4>(bv, be);
  if constexpr (G > 8) argmax_step<8>(bv, be);
  if constexpr (G > 16) argmax_step<16>(bv, be);
  if constexpr (G > 32) argmax_step<32>(bv, be);
}

// The decisions of one token, taken by its group of G lanes on v[vi] = logit of expert gl + G vi (-inf past E; consumed).
// Slot vi of lane gl receives choice j = gl + G vi: si = expert, sw = its softmax probability (not yet renormalised);
// denom = the sum of the k probabilities.  With `check` the k + 1 largest values are ordered and the result says whether
// some pair of neighbours is closer than `tol2` (twice the error bound of the logits) plus rounding slack (two units in
// the last place of the larger one); theta = the smallest value looked at.
template <int G, int V>
__device__ __forceinline__ bool token_topk(float (&v)[V], int gl, int E, int k, bool check, float tol2, int (&si)[V], float (&sw)[V],
                                           float& denom, float& theta) {
  const float NEG_INF = -__builtin_inff();
  float mx = v[0];
#pragma unroll
  for (int vi = 1; vi < V; ++vi) mx = fmaxf(mx, v[vi]);
  mx = group_max<G>(mx);
  float se = 0.f;
#pragma unroll
  for (int vi = 0; vi < V; ++vi) se += expf(v[vi] - mx);
  se = group_sum<G>(se);
#pragma unroll
  for (int vi = 0; vi < V; ++vi) { si[vi] = 0; sw[vi] = 0.f; }
  denom = 0.f;
  bool close = false;
  float prev = 0.f;
  const int rounds = (check && k < E) ? k + 1 : k;
  for (int j = 0; j < rounds; ++j) {
    float bv = v[0];
    int be = gl;
#pragma unroll
    for (int vi = 1; vi < V; ++vi)
      if (v[vi] > bv) { bv = v[vi]; be = gl + G * vi; }
    group_argmax<G>(bv, be);
    be = be < E ? be : E - 1;                          // only reachable with non-finite logits; keeps indices in range
    if (check && j > 0) close = close || !(prev - bv > tol2 + 4.8e-7f * fmaxf(fabsf(prev), fabsf(bv)));
    prev = bv;
    theta = bv;
#pragma unroll
    for (int vi = 0; vi < V; ++vi)
      if (be == gl + G * vi) v[vi] = NEG_INF;          // the chosen expert leaves the pool
    if (j < k) {
      const float pj = expf(bv - mx) / se;
      denom += pj;
#pragma unroll
      for (int vi = 0; vi < V; ++vi)
        if (j == gl + G * vi) { si[vi] = be; sw[vi] = pj; }
    }
  }
  return close;
}

// The ballot of a predicate over this lane's group of G lanes (G = 16: four groups per wave; G = 64: the wave)
template <int G> __device__ __forceinline__ unsigned long long group_ballot(bool p, int grp) {
  const unsigned long long b = __ballot(p);
  return G == 64 ? b : (b >> (G * grp)) & ((1ull << (G & 63)) - 1ull);
}

// sum over m of x[t, m] * Wt[e, m] in fp64 by a group of G lanes, for two experts at once (every product of two bf16
// values is exact in fp32; lane gl adds the 16-byte pieces gl, gl + G, ... in ascending order, then a fixed butterfly adds
// the G partial sums); all lanes of the group get both sums.  Four pieces are fetched per round so that their latencies
// overlap.
template <int G>
__device__ __forceinline__ void group_dot2_fp64(const uint16_t* __restrict__ xr, const uint16_t* __restrict__ wa,
                                                const uint16_t* __restrict__ wb, int M, int gl, double& sa, double& sb) {
  double acc_a = 0.0, acc_b = 0.0;
  const int pieces = M >> 3;
  for (int p0 = 0; p0 < pieces; p0 += 4 * G) {
    uint4 xv[4], av[4], bv[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int p = p0 + G * u + gl;
      const int q = p < pieces ? p : 0;                  // pieces past the row's end re-read its start and are zeroed
      xv[u] = *reinterpret_cast<const uint4*>(xr + q * 8);
      av[u] = *reinterpret_cast<const uint4*>(wa + q * 8);
      bv[u] = *reinterpret_cast<const uint4*>(wb + q * 8);
      if (p >= pieces) xv[u] = make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t xa[4] = {xv[u].x, xv[u].y, xv[u].z, xv[u].w};
      const uint32_t aa[4] = {av[u].x, av[u].y, av[u].z, av[u].w};
      const uint32_t ba[4] = {bv[u].x, bv[u].y, bv[u].z, bv[u].w};
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const float xl = __uint_as_float(xa[q] << 16), xh = __uint_as_float(xa[q] & 0xffff0000u);
        acc_a += (double)(xl * __uint_as_float(aa[q] << 16));
        acc_a += (double)(xh * __uint_as_float(aa[q] & 0xffff0000u));
        acc_b += (double)(xl * __uint_as_float(ba[q] << 16));
        acc_b += (double)(xh * __uint_as_float(ba[q] & 0xffff0000u));
      }
    }
  }
#pragma unroll
  for (int d = G / 2; d >= 1; d >>= 1) {
    acc_a += __shfl_xor(acc_a, d, 64);
    acc_b += __shfl_xor(acc_b, d, 64);
  }
  sa = acc_a;
  sb = acc_b;
}

// Exact decisions for one token whose approximate logits (within tol2 / 2 of the exactly rounded ones) left its top k
// open; run by a group of G lanes (a wave, or a quarter of one for gates of at most 128 experts: four tokens are then
// repaired side by side).  theta = the (k+1)-th largest approximate logit.  Every expert that can still reach the top k
// (approximate logit within tol2 of theta) is looked at; those that have another such expert within tol2 get their logit
// recomputed in fp64 from x and Wt and stored (an expert farther than that from every other keeps its place whatever the
// true values are); then the token is decided again on the repaired row.  hist: the block's packed arrival counters.
// `on` = this group has a token (groups without one run along with nothing to do).
template <int G>
__device__ __forceinline__ void repair_token(bool on, int64_t t, float theta, float tol2, int lane, float* __restrict__ logits,
                                             int E, int k, int normalize, int32_t* __restrict__ idx, float* __restrict__ gate_w,
                                             int* hist, const uint16_t* __restrict__ x, const uint16_t* __restrict__ Wt,
                                             const float* __restrict__ bias, int M, int Mp) {
  const float NEG_INF = -__builtin_inff();
  const int grp = lane / G, gl = lane % G;
  const float reach = theta - tol2 - 4.8e-7f * fabsf(theta);         // experts below this cannot be among the k largest
  float rv[8];
#pragma unroll
  for (int vi = 0; vi < 8; ++vi) {
    const int e = gl + G * vi;
    rv[vi] = (on && e < E) ? logits[t * E + e] : NEG_INF;
  }
  bool need[8];
#pragma unroll
  for (int vi = 0; vi < 8; ++vi) need[vi] = false;
#pragma unroll
  for (int vi = 0; vi < 8; ++vi) {
    unsigned long long todo = group_ballot<G>(on && rv[vi] >= reach, grp);
    while (todo) {
      const int l = __builtin_ctzll(todo);
      todo &= todo - 1;
      const float val = __shfl(rv[vi], grp * G + l, 64);
      bool near = false;
#pragma unroll
      for (int vj = 0; vj < 8; ++vj)
        near = near || (rv[vj] >= reach && !(vj == vi && gl == l) &&
                        fabsf(rv[vj] - val) <= tol2 + 4.8e-7f * fmaxf(fabsf(rv[vj]), fabsf(val)));
      if (group_ballot<G>(near, grp) != 0ull && gl == l) need[vi] = true;
    }
  }
  // the marked experts, two at a time (one pending until its partner turns up)
  const uint16_t* xr = x + (on ? t : 0) * (int64_t)M;
  int pend_e = -1, pend_l = 0, pend_vi = 0;
  auto put = [&](int e, int l, int vi, double sum) __attribute__((always_inline)) {
    const float val = (float)(sum + (bias ? (double)bias[e] : 0.0));
#pragma unroll
    for (int vj = 0; vj < 8; ++vj)
      if (vj == vi && gl == l) rv[vj] = val;
    if (gl == l) logits[t * E + e] = val;
  };
#pragma unroll
  for (int vi = 0; vi < 8; ++vi) {
    unsigned long long todo = group_ballot<G>(need[vi], grp);
    while (todo) {
      const int l = __builtin_ctzll(todo);
      todo &= todo - 1;
      const int e = l + G * vi;
      if (pend_e < 0) { pend_e = e; pend_l = l; pend_vi = vi; continue; }
      double sa, sb;
      group_dot2_fp64<G>(xr, Wt + (int64_t)pend_e * Mp, Wt + (int64_t)e * Mp, M, gl, sa, sb);
      put(pend_e, pend_l, pend_vi, sa);
      put(e, l, vi, sb);
      pend_e = -1;
    }
  }
  if (pend_e >= 0) {
    double sa, sb;
    group_dot2_fp64<G>(xr, Wt + (int64_t)pend_e * Mp, Wt + (int64_t)pend_e * Mp, M, gl, sa, sb);
    put(pend_e, pend_l, pend_vi, sa);
  }
  int si[8];
  float sw[8], denom, th;
  token_topk<G, 8>(rv, gl, E, k, false, 0.f, si, sw, denom, th);
  if (on) {
#pragma unroll
    for (int vi = 0; vi < 8; ++vi) {
      const int j = gl + G * vi;
      if (j < k) {
        idx[t * k + j] = si[vi];
        gate_w[t * k + j] = normalize ? sw[vi] / denom : sw[vi];
        atomicAdd(&hist[(j * E + si[vi]) >> 2], 1 << (8 * ((j * E + si[vi]) & 3)));
      }
    }
  }
}

// One block per 64 tokens (in arrival order).  Phase 1: every token's decisions from its logits.  With `margin` (the
// logits came from the fast kernel and are only known to within margin[t]) a token whose k + 1 largest logits are not
// separated by more than twice that bound is set aside.  Phase 2: one wave per token set aside repairs it (repair_token):
// the decisions then equal those taken on exactly rounded logits.  Phase 3: the block's per-(rank, expert) arrival counters go to memory.
template <int G, int V>
__global__ __launch_bounds__(1024) void gate_topk_kernel(float* __restrict__ logits, int64_t T, int E, int k,
                                                        int normalize, int32_t* __restrict__ idx,
                                                        float* __restrict__ gate_w, int32_t* __restrict__ block_counts,
                                                        int NB, const int32_t* __restrict__ perm,
                                                        const float* __restrict__ margin, const uint16_t* __restrict__ x,
                                                        const uint16_t* __restrict__ Wt, const float* __restrict__ bias,
                                                        int M, int Mp) {
  extern __shared__ int smem_i[];
  // [k][E] arrivals of this block's tokens: at most 64 each, so four 8-bit counters share a word (integer atomics on the
  // word: the sums do not depend on the order)
  int* hist = smem_i;
  const int hist_words = (k * E + 3) >> 2;
  int* aside_tok = smem_i + hist_words;                // [64] block-local tokens set aside
  float* aside_theta = reinterpret_cast<float*>(aside_tok + kGateTokensPerBlock);
  int* aside_n = aside_tok + 2 * kGateTokensPerBlock;
  for (int i = threadIdx.x; i < hist_words; i += blockDim.x) hist[i] = 0;
  if (threadIdx.x == 0) *aside_n = 0;
  __syncthreads();
  const int groups = blockDim.x / G, g = threadIdx.x / G, gl = threadIdx.x % G;   // blockDim.x is a multiple of 64 >= G
  const float NEG_INF = -__builtin_inff();
  const int passes = (kGateTokensPerBlock + groups - 1) / groups;
  for (int it = 0; it < passes; ++it) {
    const int tb = it * groups + g;                    // token of this block handled by this lane group in this pass
    const int64_t tv = (int64_t)blockIdx.x * kGateTokensPerBlock + tb;   // position in arrival order
    const bool valid = tb < kGateTokensPerBlock && tv < T;
    int64_t t = tv;                                                     // the token that arrives at that position
    if (valid && perm) { const int32_t p = perm[tv]; t = ((uint32_t)p < (uint64_t)T) ? p : tv; }   // clamp: never out of range
    float v[V];
#pragma unroll
    for (int vi = 0; vi < V; ++vi) {
      const int e = gl + G * vi;
      v[vi] = (valid && e < E) ? logits[t * E + e] : NEG_INF;
    }
    int si[V];
    float sw[V], denom, theta;
    const bool check = margin != nullptr;
    const float tol2 = (check && valid) ? 2.0f * margin[t] : 0.f;
    bool publish = valid;
    const bool close = token_topk<G, V>(v, gl, E, k, check, tol2, si, sw, denom, theta);
    if (check && valid && close) {                     // uniform over the token's lanes
      publish = false;
      if (gl == 0) {
        const int slot = atomicAdd(aside_n, 1);
        aside_tok[slot] = tb;
        aside_theta[slot] = theta;
      }
    }
    if (publish) {
#pragma unroll
      for (int vi = 0; vi < V; ++vi) {
        const int j = gl + G * vi;
        if (j < k) {
          idx[t * k + j] = si[vi];
          gate_w[t * k + j] = normalize ? sw[vi] / denom : sw[vi];
          atomicAdd(&hist[(j * E + si[vi]) >> 2], 1 << (8 * ((j * E + si[vi]) & 3)));
        }
      }
    }
  }
  __syncthreads();
  if (margin) {
    const int n_aside = *aside_n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    for (int i = wave; i < n_aside; i += nwaves)
      repair_token<64>(true, (int64_t)blockIdx.x * kGateTokensPerBlock + aside_tok[i], aside_theta[i],
                       2.0f * margin[(int64_t)blockIdx.x * kGateTokensPerBlock + aside_tok[i]], lane, logits, E, k, normalize, idx,
                       gate_w, hist, x, Wt, bias, M, Mp);
    __syncthreads();
  }
  for (int i = threadIdx.x; i < k * E; i += blockDim.x) {
    const int j = i / E, e = i % E;
    block_counts[((int64_t)e * k + j) * NB + blockIdx.x] = (hist[i >> 2] >> (8 * (i & 3))) & 0xff;
  }
}

// softmax + top-k with one lane per token, for k <= 32: the kernel of choice for wide gates.  A wave owns 64 consecutive
// tokens (one block of the arrival counters).  Its logits pass through LDS 32 experts at a time (rows padded to 33 words:
// the transposed reads are conflict-free); every lane walks its own row in ascending expert order and keeps the N = KMAX+1
// largest values seen so far, sorted, in registers: a new value moves in above every smaller one (strictly smaller: an
// equal value met later, i.e. a higher index, stays below) and the entries from there on shift down by one, so the list ends as the top k in the order the selection
// rule asks for, and its (k+1)-th entry serves the near-tie check.  The softmax denominator is kept chunk by chunk
// relative to the running maximum.  The four waves of a block work independently (no barrier).
template <int KMAX, bool VEC4>
__global__ __launch_bounds__(256) void gate_topk_lane_kernel(float* __restrict__ logits, int64_t T, int E, int k, int normalize,
                                                             int32_t* __restrict__ idx, float* __restrict__ gate_w,
                                                             int32_t* __restrict__ block_counts, int NB,
                                                             const float* __restrict__ margin, const uint16_t* __restrict__ x,
                                                             const uint16_t* __restrict__ Wt, const float* __restrict__ bias,
                                                             int M, int Mp) {
  constexpr int N = KMAX + 1, CW = 32, LDW = CW + 1;
  extern __shared__ int smem_i[];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int hist_words = (k * E + 3) >> 2;
  const int per_wave = kGateTokensPerBlock * LDW + hist_words;
  float* tile = reinterpret_cast<float*>(smem_i + wave * per_wave);   // [64 tokens][33]
  int* hist = smem_i + wave * per_wave + kGateTokensPerBlock * LDW;   // packed [k][E] arrival counters of this wave's tokens
  const int b = blockIdx.x * 4 + wave;                                // block of 64 tokens
  if (b >= NB) return;                                                // waves are independent: no barrier below
  const int64_t t0 = (int64_t)b * kGateTokensPerBlock;
  const int64_t t = t0 + lane;
  const bool valid = t < T;
  const float NEG_INF = -__builtin_inff();
  for (int i = lane; i < hist_words; i += 64) hist[i] = 0;

  float L[N];
  int I[N];
#pragma unroll
  for (int i = 0; i < N; ++i) { L[i] = NEG_INF; I[i] = 0x7fffffff; }
  float mx = NEG_INF, se = 0.f;
  for (int e0 = 0; e0 < E; e0 += CW) {
    // tile[row][c] = logits[t0 + row][e0 + c]  (-inf outside the matrix)
    if (VEC4) {                                                        // E % 4 == 0: 16-byte pieces, 8 rows x 128 bytes per load
      const int c4 = (lane & 7) * 4;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int row = (lane >> 3) + 8 * i;
        float4 v = make_float4(NEG_INF, NEG_INF, NEG_INF, NEG_INF);
        if (t0 + row < T && e0 + c4 < E) v = *reinterpret_cast<const float4*>(logits + (t0 + row) * E + e0 + c4);
        float* d = tile + row * LDW + c4;
        d[0] = v.x; d[1] = v.y; d[2] = v.z; d[3] = v.w;
      }
    } else {
      const int c = lane & 31;
#pragma unroll 8
      for (int i = 0; i < 32; ++i) {
        const int row = (lane >> 5) + 2 * i;
        tile[row * LDW + c] = (t0 + row < T && e0 + c < E) ? logits[(t0 + row) * E + e0 + c] : NEG_INF;
      }
    }
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_s_waitcnt(0xc07f);                                // lgkmcnt(0): the tile is in LDS before any lane reads it
    float row[CW];
#pragma unroll
    for (int c = 0; c < CW; ++c) row[c] = tile[lane * LDW + c];
    float cm = row[0];
#pragma unroll
    for (int c = 1; c < CW; ++c) cm = fmaxf(cm, row[c]);
    if (cm > mx) { se *= __expf(mx - cm); mx = cm; }                   // (0 * exp(-inf) = 0 on the first chunk)
#pragma unroll
    for (int c = 0; c < CW; ++c) {
      float v = row[c];
      int e = e0 + c;
      se += __expf(v - mx);
      bool g = false;                                                  // once the value has moved in, everything below shifts down
#pragma unroll
      for (int i = 0; i < N; ++i) {
        g = g || v > L[i];
        const float tv = g ? L[i] : v;
        const int ti = g ? I[i] : e;
        L[i] = g ? v : L[i];
        I[i] = g ? e : I[i];
        v = tv;
        e = ti;
      }
    }
    __builtin_amdgcn_wave_barrier();                                   // every lane has read its row before the next chunk lands
  }
  // near-tie check on the k + 1 largest
  bool close = false;
  const bool check = margin != nullptr;
  const float tol2 = (check && valid) ? 2.0f * margin[t] : 0.f;
  float theta = NEG_INF;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i < k || (i == k && k < E)) {
      theta = L[i];
      if (check && i > 0) close = close || !(L[i - 1] - L[i] > tol2 + 4.8e-7f * fmaxf(fabsf(L[i - 1]), fabsf(L[i])));
    }
  }
  const bool aside = check && valid && close;
  if (valid && !aside) {
    float p[KMAX], denom = 0.f;
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      p[j] = 0.f;
      if (j < k) { p[j] = expf(L[j] - mx) / se; denom += p[j]; }
    }
#pragma unroll
    for (int j = 0; j < KMAX; ++j) {
      if (j < k) {
        const int e = I[j] < E ? I[j] : E - 1;                         // only reachable with non-finite logits
        idx[t * k + j] = e;
        gate_w[t * k + j] = normalize ? p[j] / denom : p[j];
        atomicAdd(&hist[(j * E + e) >> 2], 1 << (8 * ((j * E + e) & 3)));
      }
    }
  }
  // the wave repairs its open tokens: four side by side, a quarter of the wave each, for gates of at most 128 experts
  // (their list goes through the tile's LDS, which is free now), one by one with the whole wave otherwise
  const unsigned long long open = __ballot(aside);
  if (open) {
    if (E <= 128) {
      int* list = reinterpret_cast<int*>(tile);
      if (aside) list[__popcll(open & ((1ull << lane) - 1ull))] = lane;
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_s_waitcnt(0xc07f);
      const int n_open = __popcll(open), grp = lane >> 4;
      for (int i0 = 0; i0 < n_open; i0 += 4) {
        const bool on = i0 + grp < n_open;
        const int src = on ? list[i0 + grp] : 0;
        repair_token<16>(on, t0 + src, __shfl(theta, src, 64), __shfl(tol2, src, 64), lane, logits, E, k, normalize, idx, gate_w, hist,
                         x, Wt, bias, M, Mp);
      }
    } else {
      unsigned long long todo = open;
      while (todo) {
        const int l = __builtin_ctzll(todo);
        todo &= todo - 1;
        repair_token<64>(true, t0 + l, __shfl(theta, l, 64), __shfl(tol2, l, 64), lane, logits, E, k, normalize, idx, gate_w, hist, x,
                         Wt, bias, M, Mp);
      }
    }
  }
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_s_waitcnt(0xc07f);
  for (int i = lane; i < k * E; i += 64) {
    const int j = i / E, e = i % E;
    block_counts[((int64_t)e * k + j) * NB + b] = (hist[i >> 2] >> (8 * (i & 3))) & 0xff;
  }
}

// One block per expert: exclusive scan of block_counts[e, (j, b)] (an expert's counters are contiguous, in arrival order
// (rank j, block b)) in place; totals -> counts[e];
// slots [min(total, C), C) of slot_src[e] are marked unfilled.
__global__ __launch_bounds__(256) void gate_scan_kernel(int32_t* __restrict__ block_counts, int L, int E, int64_t C,
                                                        int32_t* __restrict__ counts, int32_t* __restrict__ slot_src) {
  __shared__ int part[256];
  const int e = blockIdx.x, tid = threadIdx.x;
  const int per = (L + 255) / 256;
  const int start = min(tid * per, L), stop = min(start + per, L);
  int sum = 0;
  for (int i = start; i < stop; ++i) sum += block_counts[(int64_t)e * L + i];
  part[tid] = sum;
  __syncthreads();
  for (int off = 1; off < 256; off <<= 1) {            // inclusive Hillis-Steele scan of the 256 partial sums
    const int add = (tid >= off) ? part[tid - off] : 0;
    __syncthreads();
    part[tid] += add;
    __syncthreads();
  }
  int run = part[tid] - sum;
  for (int i = start; i < stop; ++i) {
    const int c = block_counts[(int64_t)e * L + i];
    block_counts[(int64_t)e * L + i] = run;
    run += c;
  }
  const int total = part[255];
  if (tid == 0) counts[e] = total;
  if (slot_src) {
    const int64_t first = total < C ? total : C;
    for (int64_t c = first + tid; c < C; c += 256) slot_src[(int64_t)e * C + c] = -1;
  }
}

// Number of lanes below this one whose token goes to the same expert: intersects, bit by bit of the expert's number, the
// ballots that agree with this lane's bit.
__device__ __forceinline__ int rank_among_lanes(int e, bool valid, int bits, int lane) {
  unsigned long long peers = __ballot(valid);
  for (int b = 0; b < bits; ++b) {
    const bool mine = (e >> b) & 1;
    const unsigned long long set = __ballot(mine);
    peers &= mine ? set : ~set;
  }
  return __popcll(peers & ((1ull << lane) - 1ull));
}

// One wave per block of 64 tokens, one lane per token: scanned offset plus the position among the block's earlier tokens
// with the same (rank, expert).
__global__ __launch_bounds__(kGateTokensPerBlock) void gate_assign_kernel(const int32_t* __restrict__ idx,
                                                                          const int32_t* __restrict__ block_off, int64_t T,
                                                                          int E, int bits, int k, int64_t C, int NB,
                                                                          int32_t* __restrict__ loc,
                                                                          int32_t* __restrict__ slot_src,
                                                                          const int32_t* __restrict__ perm) {
  const int lane = threadIdx.x;
  const int64_t tv = (int64_t)blockIdx.x * kGateTokensPerBlock + lane;   // position in arrival order
  const bool valid = tv < T;
  int64_t t = tv;
  if (valid && perm) { const int32_t p = perm[tv]; t = ((uint32_t)p < (uint64_t)T) ? p : tv; }
  for (int j = 0; j < k; ++j) {
    const int e = valid ? idx[t * k + j] : 0;
    const int r = rank_among_lanes(e, valid, bits, lane);
    if (valid) {
      const int l = block_off[((int64_t)e * k + j) * NB + blockIdx.x] + r;
      loc[t * k + j] = l;
      if (slot_src && l < C) slot_src[(int64_t)e * C + l] = (int32_t)t;
    }
  }
}

// Scan and assignment in one launch, for counters few enough that every block adds them up by itself: `before` of an (expert,
// rank) = all arrivals at lower ranks + those of this rank in earlier blocks.  Saves a launch and its wait where those are
// what the stage costs: 1 to 2 us of a small gate's 6 to 10.
__global__ __launch_bounds__(256) void gate_slots_kernel(const int32_t* __restrict__ idx, const int32_t* __restrict__ block_counts,
                                                         int64_t T, int E, int bits, int k, int64_t C, int NB,
                                                         int32_t* __restrict__ counts, int32_t* __restrict__ loc,
                                                         int32_t* __restrict__ slot_src, int mark_unfilled,
                                                         const int32_t* __restrict__ perm) {
  __shared__ int all[kSlotsMaxPairs], before[kSlotsMaxPairs];
  const int lane = threadIdx.x & 63, pairs = E * k;
  for (int q = threadIdx.x; q < pairs; q += 256) { all[q] = 0; before[q] = 0; }
  __syncthreads();
#pragma unroll 4
  for (int i = threadIdx.x; i < pairs * NB; i += 256) {             // integer sums: their order does not matter
    const int c = block_counts[i], q = i / NB, b = i - q * NB;
    if (c) {
      atomicAdd(&all[q], c);
      if (b < (int)blockIdx.x) atomicAdd(&before[q], c);
    }
  }
  __syncthreads();
  for (int e = threadIdx.x; e < E; e += 256) {                      // ranks in order: exclusive sums over the lower ones
    int run = 0;
    for (int j = 0; j < k; ++j) { before[e * k + j] += run; run += all[e * k + j]; }
    all[e * k] = run;                                               // the expert's arrivals
    if (blockIdx.x == 0) counts[e] = run;
  }
  __syncthreads();
  if (mark_unfilled && slot_src) {
    for (int e = blockIdx.x; e < E; e += gridDim.x) {
      const int64_t total = all[e * k], first = total < C ? total : C;
      for (int64_t c = first + threadIdx.x; c < C; c += 256) slot_src[(int64_t)e * C + c] = -1;
    }
  }
  if (threadIdx.x >= kGateTokensPerBlock) return;
  const int64_t tv = (int64_t)blockIdx.x * kGateTokensPerBlock + lane;
  const bool valid = tv < T;
  int64_t t = tv;
  if (valid && perm) { const int32_t p = perm[tv]; t = ((uint32_t)p < (uint64_t)T) ? p : tv; }
  for (int j = 0; j < k; ++j) {
    const int e = valid ? idx[t * k + j] : 0;
    const int r = rank_among_lanes(e, valid, bits, lane);
    if (valid) {
      const int l = before[e * k + j] + r;
      loc[t * k + j] = l;
      if (slot_src && l < C) slot_src[(int64_t)e * C + l] = (int32_t)t;
    }
  }
}

// Top-k, scan and assignment of a small gate in one launch of one block (the rule: gate_rules.h): a lane per token, a wave per 64 of
// them.  A token's E <= 16 logits and the k choices stay in its lane's registers; the decisions are those of token_topk, sums of the softmax
// in the same order.  Arrivals are counted in LDS by wave, scanned there (rank, then wave), and a lane's place
// among its wave's comes from ballots as in gate_assign_kernel.  Such a gate is launches that wait for each other, not work: captured,
// top-k on: 16 tokens, 8 experts, top-2 6.1 -> 4.9 us; 512 tokens, 4 experts, top-1 5.4 -> 2.9; 1024 tokens 5.4 -> 3.3.
template <int G>
__device__ __forceinline__ void decide_small_gate(const float* logits, int T, int E, int bits, int k, int64_t C, int normalize, int32_t* __restrict__ idx,
                                                  float* __restrict__ gate_w, int32_t* __restrict__ loc, int32_t* __restrict__ counts,
                                                  int32_t* __restrict__ slot_src, int mark_unfilled, const int32_t* __restrict__ perm) {
  constexpr int W = kSmallGateTokens / kWave;
  // pairs and choices that the rule lets in, with more than G / 2 experts
  constexpr int P = G * G < kSmallGatePairs ? G * G : kSmallGatePairs, R = kSmallGatePairs / (G / 2 + 1) < G ? kSmallGatePairs / (G / 2 + 1) : G;
  __shared__ int cnt[P][W + 1], total[P];                           // [expert * k + rank]: arrivals by wave, then of earlier waves
  __shared__ float prob[R][kSmallGateTokens];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, tv = (int)threadIdx.x, pairs = E * k;
  const int waves = (int)blockDim.x >> 6;
  const bool valid = tv < T;
  int t = valid ? tv : 0;                                           // the token that arrives at position tv
  if (valid && perm) { const int32_t p = perm[tv]; t = (uint32_t)p < (uint32_t)T ? p : tv; }
  const float NEG_INF = -__builtin_inff();
  float v[G];
  const float* row = logits + (int64_t)t * E;
  if (E == G && G % 4 == 0 && ((uintptr_t)logits & 15) == 0) {
#pragma unroll
    for (int e = 0; e + 3 < G; e += 4) {
      const float4 q = *reinterpret_cast<const float4*>(row + e);
      v[e] = q.x; v[e + 1] = q.y; v[e + 2] = q.z; v[e + 3] = q.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < G; ++e) v[e] = row[e < E ? e : 0];
  }
#pragma unroll
  for (int e = 0; e < G; ++e) v[e] = valid && e < E ? v[e] : NEG_INF;
  for (int i = threadIdx.x; i < pairs * W; i += blockDim.x) cnt[i / W][i % W] = 0;
  __syncthreads();
  float mx = v[0];
#pragma unroll
  for (int e = 1; e < G; ++e) mx = fmaxf(mx, v[e]);
  float s[G];
#pragma unroll
  for (int e = 0; e < G; ++e) s[e] = expf(v[e] - mx);
#pragma unroll
  for (int d = 1; d < G; d <<= 1)
#pragma unroll
    for (int e = 0; e < G; e += 2 * d) s[e] += s[e + d];
  // choices: four bits each; their probabilities go to LDS.  One body for every rank: this kernel runs for so
  // short a time that fetching its code is part of it (and a row comes in 16-byte pieces: 64 tokens, 16 experts,
  // top-1 5.8 us, 8.8 with coalesced loads through LDS, whose indexes take divisions).
  uint64_t chosen = 0;
  float denom = 0.f;
#pragma unroll 1
  for (int j = 0; j < k; ++j) {
    float bv = v[0];
    int be = 0;
#pragma unroll
    for (int e = 1; e < G; ++e)
      if (v[e] > bv) { bv = v[e]; be = e; }
    be = be < E ? be : E - 1;                                       // only reachable with non-finite logits
#pragma unroll
    for (int e = 0; e < G; ++e)
      if (be == e) v[e] = NEG_INF;                                  // the chosen expert leaves the pool
    const float pj = expf(bv - mx) / s[0];
    denom += pj;
    prob[j][tv] = pj;
    chosen |= (uint64_t)be << (4 * j);
    if (valid) atomicAdd(&cnt[be * k + j][wave], 1);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < pairs; q += blockDim.x) {
    int run = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const int c = cnt[q][w];
      cnt[q][w] = run;
      run += c;
    }
    total[q] = run;
  }
  __syncthreads();
#pragma unroll 1
  for (int j = 0; j < k; ++j) {
    const int e = (int)(chosen >> (4 * j)) & 15, r = rank_among_lanes(e, valid, bits, lane);
    if (valid) {
      int l = cnt[e * k + j][wave] + r;
      for (int i = 0; i < j; ++i) l += total[e * k + i];
      const float pj = prob[j][tv];
      idx[t * k + j] = e;
      gate_w[t * k + j] = normalize ? pj / denom : pj;
      loc[t * k + j] = l;
      if (slot_src && l < C) slot_src[(int64_t)e * C + l] = t;
    }
  }
  for (int e = wave; e < E; e += waves) {
    int64_t n = 0;
    for (int j = 0; j < k; ++j) n += total[e * k + j];
    if (lane == 0) counts[e] = (int32_t)n;
    if (mark_unfilled && slot_src)
      for (int64_t c = (n < C ? n : C) + lane; c < C; c += kWave) slot_src[(int64_t)e * C + c] = -1;
  }
}

template <int G>
__global__ __launch_bounds__(kSmallGateTokens) void gate_small_kernel(const float* __restrict__ logits, int T, int E, int bits, int k, int64_t C,
                                                                      int normalize, int32_t* __restrict__ idx, float* __restrict__ gate_w,
                                                                      int32_t* __restrict__ loc, int32_t* __restrict__ counts,
                                                                      int32_t* __restrict__ slot_src, int mark_unfilled,
                                                                      const int32_t* __restrict__ perm) {
  decide_small_gate<G>(logits, T, E, bits, k, C, normalize, idx, gate_w, loc, counts, slot_src, mark_unfilled, perm);
}

// The whole gate of up to 16 tokens (the rule: gate_rules.h): the one tile of logits_of_tiles and, in the same block, the decisions on it.  A decode step
// is launches that wait for each other: logits 8.2 us and decisions 4.9 in two launches, 12.3 so by the profiler, and a launch less to wait for (16 tokens, 8 experts
// 2048 x 2048, whole pass 47.4 -> 46.0; 256 x 256, 4 experts 19.0 -> 17.1).  Of the 12 us 5.9 do not depend on M (launch, the sums through LDS, the decisions, their stores: captured, M = 8),
// and each 1024 k are another 2.9, of which one unit's fp64 matrix pipes take 1.7 (M / 4 instructions of 64 cycles over four of them at 2.4 GHz) and the passes' trips to memory the
// rest; with four passes in flight instead of two 12.8.
template <typename XT, int G>
__global__ __launch_bounds__(64 * 16) void gate_few_tokens_kernel(const XT* __restrict__ x, const XT* __restrict__ Wg, const float* __restrict__ bias, int T,
                                                                  int M, int E, float* logits, int bits, int k, int64_t C, int normalize,
                                                                  int32_t* __restrict__ idx, float* __restrict__ gate_w, int32_t* __restrict__ loc,
                                                                  int32_t* __restrict__ counts, int32_t* __restrict__ slot_src, int mark_unfilled) {
  logits_of_tiles<XT, 1, 16, 1>(x, Wg, bias, T, M, E, 0, 0, logits);
  __syncthreads();
  decide_small_gate<G>(logits, T, E, bits, k, C, normalize, idx, gate_w, loc, counts, slot_src, mark_unfilled, nullptr);
}

hipError_t launch_gate_few_tokens(const void* x, const void* Wg, const float* bias, int dtype, int64_t T, int64_t M, int64_t E, float* logits, int k,
                                  int64_t C, int normalize, int32_t* idx, float* gate_w, int32_t* loc, int32_t* counts, int32_t* slot_src,
                                  bool mark_unfilled, hipStream_t s) {
  int bits = 0;
  while ((1 << bits) < E) ++bits;
#define MOE_FEW(XT, GG)                                                                                                                   \
  gate_few_tokens_kernel<XT, GG><<<dim3(1), dim3(64 * 16), 0, s>>>((const XT*)x, (const XT*)Wg, bias, (int)T, (int)M, (int)E, logits, bits, k, C, \
                                                                   normalize, idx, gate_w, loc, counts, slot_src, mark_unfilled)
#define MOE_FEW_G(XT)                 \
  do {                                \
    if (E <= 4) MOE_FEW(XT, 4);       \
    else if (E <= 8) MOE_FEW(XT, 8);  \
    else MOE_FEW(XT, 16);             \
  } while (0)
  if (dtype == MOE_F32) MOE_FEW_G(float);
  else MOE_FEW_G(uint16_t);
#undef MOE_FEW_G
#undef MOE_FEW
  return hipGetLastError();
}

hipError_t launch_gate_topk(float* logits, int64_t T, int64_t E, int k, int64_t C, int normalize, int32_t* idx,
                            float* gate_w, int32_t* loc, int32_t* counts, int32_t* slot_src, int32_t* block_counts,
                            hipStream_t s, const int32_t* perm, const GateRepair* repair, bool mark_unfilled) {
  const int NB = (int)ceil_div(T, kGateTokensPerBlock);
  // lane group per token: up to 16 experts one value per lane; from there on 16 lanes with up to 8 logits each (4 tokens
  // per wave), and a whole wave beyond 128 experts
  int G = 1;
  while (G < E && G < 16) G <<= 1;
  if (E > 128) G = 64;
  int bits = 0;
  while ((1 << bits) < E) ++bits;
  if (!repair && gate_in_one_block(T, E, k, slot_src && mark_unfilled ? C : 0)) {
    const dim3 all((unsigned)(ceil_div(T, kWave) * kWave));
#define MOE_SMALL(GG) gate_small_kernel<GG><<<dim3(1), all, 0, s>>>(logits, (int)T, (int)E, bits, k, C, normalize, idx, gate_w, loc, counts, slot_src, mark_unfilled, perm)
    if (G == 1) MOE_SMALL(1);
    else if (G == 2) MOE_SMALL(2);
    else if (G == 4) MOE_SMALL(4);
    else if (G == 8) MOE_SMALL(8);
    else MOE_SMALL(16);
#undef MOE_SMALL
    return hipGetLastError();
  }
  const int V = (int)ceil_div(E, G);
  const size_t shmem = (((size_t)k * E + 3) / 4 + 2 * kGateTokensPerBlock + 1) * sizeof(int);
  // one lane group per token: as many threads as the block's 64 tokens need, so that (up to 16 experts) every token's
  // logits are fetched in one round instead of one dependent round trip per pass
  const dim3 grid(NB), block(256);
  const dim3 tblock((unsigned)(64 * G < 256 ? 256 : (64 * G > 1024 ? 1024 : 64 * G)));
  const float* margin = repair ? repair->margin : nullptr;
  const uint16_t* rx = repair ? (const uint16_t*)repair->x : nullptr;
  const uint16_t* rw = repair ? repair->Wt : nullptr;
  const float* rb = repair ? repair->bias : nullptr;
  const int rM = repair ? (int)repair->M : 0, rMp = repair ? (int)repair->Mp : 0;
#define MOE_TOPK(GG, VV) gate_topk_kernel<GG, VV><<<grid, tblock, shmem, s>>>(logits, T, (int)E, k, normalize, idx, gate_w, block_counts, NB, perm, margin, rx, rw, rb, rM, rMp)
#define MOE_TOPK_LANE(KM)                                                                                                     \
  do {                                                                                                                        \
    const size_t lsh = 4 * ((size_t)kGateTokensPerBlock * 33 + ((size_t)k * E + 3) / 4) * sizeof(int);                        \
    const dim3 lgrid((unsigned)ceil_div(NB, 4));                                                                              \
    if (E % 4 == 0) gate_topk_lane_kernel<KM, true><<<lgrid, block, lsh, s>>>(logits, T, (int)E, k, normalize, idx, gate_w, block_counts, NB, margin, rx, rw, rb, rM, rMp); \
    else gate_topk_lane_kernel<KM, false><<<lgrid, block, lsh, s>>>(logits, T, (int)E, k, normalize, idx, gate_w, block_counts, NB, margin, rx, rw, rb, rM, rMp); \
  } while (0)
  // wide gates with few choices: one lane per token (its LDS footprint, 4 waves x (8.25 KB + k E bytes), must fit 64 KB);
  // tokens in a caller-given order (perm) keep the lane-group kernel
  const bool lane_kernel = !perm && NB >= gate_lane_topk_blocks(E, k, repair ? repair->M : 0) && E > 16 && k <= 32 && (size_t)k * E <= 7936;
  if (lane_kernel) {
    if (k <= 1) MOE_TOPK_LANE(1); else if (k <= 2) MOE_TOPK_LANE(2); else if (k <= 4) MOE_TOPK_LANE(4);
    else if (k <= 8) MOE_TOPK_LANE(8); else if (k <= 16) MOE_TOPK_LANE(16); else MOE_TOPK_LANE(32);
  }
  else if (G == 1) MOE_TOPK(1, 1);
  else if (G == 2) MOE_TOPK(2, 1);
  else if (G == 4) MOE_TOPK(4, 1);
  else if (G == 8) MOE_TOPK(8, 1);
  else if (G == 16) { if (V == 1) MOE_TOPK(16, 1); else if (V == 2) MOE_TOPK(16, 2); else if (V <= 4) MOE_TOPK(16, 4); else MOE_TOPK(16, 8); }
  else { if (V <= 4) MOE_TOPK(64, 4); else MOE_TOPK(64, 8); }
#undef MOE_TOPK
#undef MOE_TOPK_LANE
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (slots_in_one_launch(NB, E, k)) {
    gate_slots_kernel<<<grid, block, 0, s>>>(idx, block_counts, T, (int)E, bits, k, C, NB, counts, loc, slot_src, mark_unfilled, perm);
    return hipGetLastError();
  }
  gate_scan_kernel<<<dim3((unsigned)E), block, 0, s>>>(block_counts, k * NB, (int)E, C, counts, mark_unfilled ? slot_src : nullptr);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  gate_assign_kernel<<<grid, dim3(kGateTokensPerBlock), 0, s>>>(idx, block_counts, T, (int)E, bits, k, C, NB, loc, slot_src, perm);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Dynamic capacity factor (Sec. 4.1): out[0] = capacity to use, out[1] = needed capacity = max_e counts[e].
// bound > 0: capacity that the factor's upper bound gives (setting < 0); bound = 0: no upper bound (setting = 0).
// ---------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dynamic_capacity_kernel(const int32_t* __restrict__ counts, int E, int64_t bound,
                                                               int64_t fixed, int64_t* __restrict__ out,
                                                               int32_t* __restrict__ fills) {
  // fixed > 0: that capacity whatever the arrivals are (a static factor); else the needed capacity, at most `bound`
  // (if bound > 0).  fills (optional): min(counts[e], chosen capacity) per expert.
  __shared__ int part[4];
  __shared__ int64_t chosen;
  int m = 0;
  for (int e = threadIdx.x; e < E; e += 256) m = max(m, counts[e]);
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) m = max(m, __shfl_xor(m, d, 64));
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    const int64_t needed = max(max(part[0], part[1]), max(part[2], part[3]));
    int64_t C = fixed > 0 ? fixed : needed;
    if (bound > 0 && C > bound) C = bound;
    if (C < 1) C = 1;                                   // an empty layer still has one (unfilled) slot per expert
    out[0] = C;
    out[1] = needed;
    chosen = C;
  }
  __syncthreads();
  if (fills) {
    const int64_t C = chosen;
    for (int e = threadIdx.x; e < E; e += 256) {
      const int64_t c = counts[e];
      fills[e] = (int32_t)(c < C ? (c > 0 ? c : 0) : C);
    }
  }
}

hipError_t launch_dynamic_capacity(const int32_t* counts, int64_t E, int64_t bound, int64_t* out, hipStream_t s,
                                   int64_t fixed, int32_t* fills) {
  dynamic_capacity_kernel<<<dim3(1), dim3(256), 0, s>>>(counts, (int)E, bound, fixed, out, fills);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// slot_src[e,c] for a capacity chosen after the arrivals were counted: -1 everywhere, then every kept choice writes
// its token (loc is unique per expert, so no two writes meet).
// ---------------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void fill_i32_kernel(int32_t* __restrict__ p, int64_t n, int32_t v) {
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) p[i] = v;
}

__global__ __launch_bounds__(256) void slot_sources_kernel(const int32_t* __restrict__ idx, const int32_t* __restrict__ loc,
                                                           int64_t pairs, int k, int E, int64_t C, int32_t* __restrict__ slot_src) {
  for (int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x; p < pairs; p += (int64_t)gridDim.x * 256) {
    const int e = idx[p], l = loc[p];
    if (l >= 0 && l < C && (unsigned)e < (unsigned)E) slot_src[(int64_t)e * C + l] = (int32_t)(p / k);
  }
}

hipError_t launch_slot_sources(const int32_t* idx, const int32_t* loc, int64_t T, int64_t E, int k, int64_t C,
                               int32_t* slot_src, hipStream_t s) {
  const int64_t n = E * C, fb = ceil_div(n, 256 * 4);
  fill_i32_kernel<<<dim3((unsigned)(fb < 8192 ? fb : 8192)), dim3(256), 0, s>>>(slot_src, n, -1);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  const int64_t pairs = T * k, sb = ceil_div(pairs, 256);
  slot_sources_kernel<<<dim3((unsigned)(sb < 8192 ? sb : 8192)), dim3(256), 0, s>>>(idx, loc, pairs, k, (int)E, C, slot_src);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Cosine router (Appendix, "A New Cosine Router"): logits[t,e] = cos(W x_t, M_e) / tau.  The projection W x runs on the
// fp64 matrix-core kernel above (rounded once to fp32); the cosine itself is a handful of fp64 operations per pair.
// ---------------------------------------------------------------------------------------------------------------
// One block per expert: MeT[d][e] = Me[e][d] widened to fp64, norm[e] = max(||Me[e]||, 1e-12).
__global__ __launch_bounds__(256) void cosine_prepare_kernel(const float* __restrict__ Me, int E, int D,
                                                             double* __restrict__ MeT, double* __restrict__ norm) {
  __shared__ double part[256];
  const int e = blockIdx.x;
  double s = 0.0;
  for (int d = threadIdx.x; d < D; d += 256) {
    const double v = (double)Me[(int64_t)e * D + d];
    MeT[(int64_t)d * E + e] = v;
    s += v * v;
  }
  part[threadIdx.x] = s;
  __syncthreads();
  for (int off = 128; off >= 1; off >>= 1) {              // fixed tree: the same sum on every run
    if (threadIdx.x < off) part[threadIdx.x] += part[threadIdx.x + off];
    __syncthreads();
  }
  if (threadIdx.x == 0) norm[e] = fmax(sqrt(part[0]), 1e-12);
}

// A wave owns 16 tokens and NT tiles of 16 experts on the fp64 matrix cores; a block's four waves share the experts.  The
// projections (as fp32) and the experts' vectors pass through LDS 32 dimensions at a time, the next ones fetched to
// registers meanwhile, so every global access is contiguous and any D works.  The squared norms come from the same operand
// values.  Bound by the latency of D / 32 rounds; one lane per expert and a broadcast per dimension, which this replaced, was
// a serial chain of 2 D fp64 operations with half the lanes idle at 32 experts: 25088 tokens, D = 256, 214 -> 19 us.
template <int NT>
__global__ __launch_bounds__(256) void cosine_logits_kernel(const float* __restrict__ proj, const double* __restrict__ MeT,
                                                            const double* __restrict__ norm, double tau, int64_t T, int D,
                                                            int E, int expert_blocks, float* __restrict__ logits) {
  constexpr int EN = NT * 16, DK = 32;
  constexpr int LDP = 36, LDM = NT == 1 ? EN : EN + 16;             // the rows of an operand read lie in different banks
  constexpr int WPT = DK * EN / 256;
  __shared__ float ps[64 * LDP];
  __shared__ double ms[DK * LDM];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r = lane & 15, kq = lane >> 4;
  const int64_t t0 = (int64_t)(blockIdx.x / expert_blocks) * 64;
  const int e0 = (int)(blockIdx.x % expert_blocks) * EN;
  float pr[8];                                                      // thread i: dimension i % 32 of tokens i / 32 + 8 u
  double mr[WPT];                                                   // and pieces i + 256 u of the [32][EN] chunk
  auto fetch = [&](int d0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int64_t t = t0 + (threadIdx.x >> 5) + 8 * u;
      const int d = d0 + (threadIdx.x & 31);
      const float v = proj[(t < T ? t : T - 1) * D + (d < D ? d : 0)];
      pr[u] = d < D ? v : 0.f;
    }
#pragma unroll
    for (int u = 0; u < WPT; ++u) {
      const int id = threadIdx.x + 256 * u, d = d0 + id / EN, e = e0 + id % EN;
      const double v = MeT[(int64_t)(d < D ? d : 0) * E + (e < E ? e : E - 1)];
      mr[u] = d < D ? v : 0.0;                                      // experts past the last repeat it and are never stored
    }
  };
  f64x4 acc[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) acc[nt] = f64x4{0.0, 0.0, 0.0, 0.0};
  double n2 = 0.0;                                                  // this lane's share of token r's squared norm
  fetch(0);
  for (int d0 = 0; d0 < D; d0 += DK) {
    __syncthreads();
#pragma unroll
    for (int u = 0; u < 8; ++u) ps[((threadIdx.x >> 5) + 8 * u) * LDP + (threadIdx.x & 31)] = pr[u];
#pragma unroll
    for (int u = 0; u < WPT; ++u) ms[((threadIdx.x + 256 * u) / EN) * LDM + (threadIdx.x + 256 * u) % EN] = mr[u];
    __syncthreads();
    if (d0 + DK < D) fetch(d0 + DK);
#pragma unroll
    for (int s = 0; s < DK / 4; ++s) {
      const double a = (double)ps[(wave * 16 + r) * LDP + 4 * s + kq];
      n2 = fma(a, a, n2);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
        acc[nt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, ms[(4 * s + kq) * LDM + nt * 16 + r], acc[nt], 0, 0, 0);
    }
  }
  n2 += __shfl_xor(n2, 16, 64);
  n2 += __shfl_xor(n2, 32, 64);                                     // now the whole norm of token r
  const double nt_own = fmax(sqrt(n2), 1e-12);
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const double nx = __shfl(nt_own, 4 * v + kq, 64);               // of the token this register belongs to
    const int64_t t = t0 + wave * 16 + 4 * v + kq;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const int e = e0 + nt * 16 + r;
      if (e < E && t < T) logits[t * E + e] = (float)((acc[nt][v] / (nx * norm[e])) / tau);
    }
  }
}

hipError_t launch_gate_logits_cosine(const void* x, const void* Wp, const float* Me, double tau, int dtype, int64_t T,
                                     int64_t M, int64_t D, int64_t E, float* logits, float* proj, double* MeT, double* norm,
                                     hipStream_t s) {
  hipError_t err = launch_gate_logits(x, Wp, nullptr, dtype, T, M, D, proj, s);
  if (err != hipSuccess) return err;
  cosine_prepare_kernel<<<dim3((unsigned)E), dim3(256), 0, s>>>(Me, (int)E, (int)D, MeT, norm);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  constexpr int64_t most = (int64_t)1 << 26;                         // tokens to a launch: at most 2^20 blocks x 8 x 256 threads
#define MOE_COSINE(NT)                                                                                                        \
  do {                                                                                                                        \
    const int64_t eb = ceil_div(E, NT * 16);                                                                                  \
    for (int64_t t = 0; t < T; t += most) {                                                                                   \
      const int64_t n = T - t < most ? T - t : most;                                                                          \
      cosine_logits_kernel<NT><<<dim3((unsigned)(ceil_div(n, 64) * eb)), dim3(256), 0, s>>>(proj + t * D, MeT, norm, tau, n, (int)D, (int)E, (int)eb, logits + t * E); \
    }                                                                                                                         \
  } while (0)
  if (E <= 16) MOE_COSINE(1); else if (E <= 32) MOE_COSINE(2); else MOE_COSINE(4);
#undef MOE_COSINE
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------------------------
// Batch prioritized routing (named in Sec. 3.2 and the Appendix's routing ablation): tokens take their slots in order
// of decreasing priority, priority = the token's largest routing probability 1 / sum_e exp(l_e - l_max), computed in
// fp64 and rounded to fp32 so that the order is a decision on an exactly comparable key; ties -> lower token.
// ---------------------------------------------------------------------------------------------------------------
// The sort key ascends as the fp32 priority descends.  A priority lies in [1/512, 1] (its sum has one to 512 terms, the largest
// of them 1), so 27 bits tell all of them apart; tokens with a NaN among their logits come first (negative NaNs before
// positive ones, as their bit patterns order).  A stable sort keeps equal priorities in token order.
//
// Stable least-significant-digit radix sort of (key, token) pairs, three passes of 9 bits and four launches in all:
//   bpr_key_kernel   : keys, and the first digit's histogram of every quarter tile
//   bpr_sort_kernel  : one pass.  A block owns a tile of consecutive pairs; it adds up the histograms of all tiles (at most
//                      128 x 512 counters) and of those before its own by itself instead of waiting for a scan, ranks its
//                      pairs (a pair's place = start of its (digit, tile) run + the pairs of that digit before it in the
//                      tile), moves them and counts the next digit of every pair into the histogram of the tile it lands in.
// Integer sums only (the atomics' order does not matter); every result is a pure function of the keys.  A chain of small
// launches, bound by their number and latency: digits of 11, 11 and 10 bits over tiles of 2048 pairs with a histogram, a
// one-block scan and a scatter launch each took ten launches, 25088 tokens 120 us; now 34 us.
constexpr int kSortBits = 9, kSortBins = 1 << kSortBits, kSortSub = 1024, kSortMaxTiles = 128;
inline int64_t sort_subs(int64_t T) { return ceil_div(T, (int64_t)kSortSub * kSortMaxTiles); }   // tiles are this many times 1024 pairs

__device__ __forceinline__ uint32_t bpr_key(float prio) {
  const uint32_t b = __float_as_uint(prio);
  const uint32_t one = 0x3F800000u, least = 0x3B000000u;            // 1 and 1/512
  return b >= least && b <= one ? one - b + 2u : (b >> 31 ? 0u : 1u);
}

// A block owns subs x 256 consecutive tokens (a quarter of a tile).  hist0[block][digit] is written whole; hist1 and hist2
// ([tiles][digits], `clear` counters in all) are cleared for the atomics of the passes.
template <bool VEC4>
__global__ __launch_bounds__(256) void bpr_key_kernel(const float* __restrict__ logits, int64_t T, int E, int subs,
                                                      uint32_t* __restrict__ key, int32_t* __restrict__ val,
                                                      uint32_t* __restrict__ hist0, uint32_t* __restrict__ hist12, int64_t clear) {
  __shared__ uint32_t h[kSortBins];
  for (int i = threadIdx.x; i < kSortBins; i += 256) h[i] = 0;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < clear; i += (int64_t)gridDim.x * 256) hist12[i] = 0;
  __syncthreads();
  for (int q = 0; q < subs; ++q) {
    const int64_t t = ((int64_t)blockIdx.x * subs + q) * 256 + threadIdx.x;
    if (t >= T) break;
    const float* row = logits + t * E;
    float mx = row[0];
    double se = 0.0;
    if (VEC4) {                                                     // rows are 16-byte aligned; the same sums in the same order
#pragma unroll 4
      for (int e = 0; e < E; e += 4) {
        const float4 v = *reinterpret_cast<const float4*>(row + e);
        mx = fmaxf(fmaxf(fmaxf(fmaxf(mx, v.x), v.y), v.z), v.w);
      }
#pragma unroll 4
      for (int e = 0; e < E; e += 4) {
        const float4 v = *reinterpret_cast<const float4*>(row + e);
        se += exp((double)v.x - (double)mx);
        se += exp((double)v.y - (double)mx);
        se += exp((double)v.z - (double)mx);
        se += exp((double)v.w - (double)mx);
      }
    } else {
      for (int e = 1; e < E; ++e) mx = fmaxf(mx, row[e]);
      for (int e = 0; e < E; ++e) se += exp((double)row[e] - (double)mx);
    }
    const uint32_t k = bpr_key((float)(1.0 / se));
    key[t] = k;
    val[t] = (int32_t)t;
    atomicAdd(&h[k & (kSortBins - 1)], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kSortBins; i += 256) hist0[(int64_t)blockIdx.x * kSortBins + i] = h[i];
}

// hist: [rows][digits] of this pass, `rows_per_tile` rows to a tile.  hist_next (optional): [tiles][digits] of the next digit.
__global__ __launch_bounds__(1024) void bpr_sort_kernel(const uint32_t* __restrict__ key_in, const int32_t* __restrict__ val_in,
                                                        int64_t n, int subs, int shift, const uint32_t* __restrict__ hist, int rows,
                                                        int rows_per_tile, uint32_t* __restrict__ hist_next,
                                                        uint32_t* __restrict__ key_out, int32_t* __restrict__ val_out) {
  constexpr int NW = 16;
  __shared__ uint32_t start[kSortBins];                             // where this tile's run of a digit begins
  __shared__ uint32_t half_all[kSortBins], half_before[kSortBins], wave_tot[8];
  __shared__ uint16_t cnt[NW][kSortBins];                           // pairs of each digit in each wave, then in the waves before it
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int d_own = threadIdx.x & (kSortBins - 1), half = threadIdx.x >> kSortBits;
  {                                                                 // totals of a digit: even rows by one half of the block, odd by the other
    const int first = blockIdx.x * rows_per_tile;
    uint32_t all = 0, before = 0;
#pragma unroll 8
    for (int r = half; r < rows; r += 2) {
      const uint32_t c = hist[(int64_t)r * kSortBins + d_own];
      all += c;
      before += r < first ? c : 0u;
    }
    if (half == 1) { half_all[d_own] = all; half_before[d_own] = before; }
    __syncthreads();
    uint32_t inc = 0;
    if (half == 0) {                                                // waves 0 .. 7: scan over the digits
      all += half_all[d_own];
      before += half_before[d_own];
      inc = all;
#pragma unroll
      for (int s = 1; s < 64; s <<= 1) {
        const uint32_t v = __shfl_up(inc, s, 64);
        if (lane >= s) inc += v;
      }
      if (lane == 63) wave_tot[wave] = inc;
    }
    __syncthreads();
    if (half == 0) {
      uint32_t base = inc - all + before;
      for (int w = 0; w < wave; ++w) base += wave_tot[w];
      start[d_own] = base;
    }
  }
  const int64_t tile_pairs = (int64_t)subs * kSortSub;
  for (int q = 0; q < subs; ++q) {                                  // 1024 pairs at a time, in order
    for (int i = threadIdx.x; i < NW * kSortBins / 2; i += 1024) reinterpret_cast<uint32_t*>(&cnt[0][0])[i] = 0;
    __syncthreads();
    const int64_t i = blockIdx.x * tile_pairs + (int64_t)q * kSortSub + threadIdx.x;
    const bool live = i < n;
    const uint32_t k = live ? key_in[i] : 0u;
    const int32_t v = live ? val_in[i] : 0;
    const int d = (int)((k >> shift) & (uint32_t)(kSortBins - 1));
    // lanes of this wave with the same digit: intersect, bit by bit, the ballots that agree with this lane's bit
    unsigned long long peers = __ballot(live);
#pragma unroll
    for (int bit = 0; bit < kSortBits; ++bit) {
      const unsigned long long set = __ballot((d >> bit) & 1);
      peers &= ((d >> bit) & 1) ? set : ~set;
    }
    const int rank_in_wave = __popcll(peers & ((1ull << lane) - 1ull));
    if (live && rank_in_wave == 0) cnt[wave][d] = (uint16_t)__popcll(peers);   // the group's first lane reports its size
    __syncthreads();
    uint32_t sum = 0;
    if (half == 0) {
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const uint32_t c = cnt[w][d_own];
        cnt[w][d_own] = (uint16_t)sum;
        sum += c;
      }
    }
    __syncthreads();
    if (live) {
      const uint32_t dst = start[d] + cnt[wave][d] + rank_in_wave;
      key_out[dst] = k;
      val_out[dst] = v;
      if (hist_next) atomicAdd(&hist_next[(int64_t)(dst / (uint32_t)tile_pairs) * kSortBins + ((k >> (shift + kSortBits)) & (kSortBins - 1))], 1u);
    }
    __syncthreads();
    if (half == 0) start[d_own] += sum;                             // read again only behind the next barrier
  }
}

size_t bpr_order_workspace_bytes(int64_t T) {
  const int64_t subs = sort_subs(T);
  const size_t rows0 = (size_t)ceil_div(T, 256 * subs), tiles = (size_t)ceil_div(T, kSortSub * subs);
  return 4 * align_up((size_t)T * 4, 256) + (rows0 + 2 * tiles) * kSortBins * 4;
}

// perm[i] = the token that arrives i-th under batch prioritized routing; returns it through *perm (a piece of ws)
hipError_t launch_bpr_order(const float* logits, int64_t T, int64_t E, void* ws, const int32_t** perm, hipStream_t s) {
  const int64_t subs = sort_subs(T);
  const int rows0 = (int)ceil_div(T, 256 * subs), tiles = (int)ceil_div(T, kSortSub * subs);
  const size_t piece = align_up((size_t)T * 4, 256);
  char* base = (char*)ws;
  uint32_t* key[2] = {(uint32_t*)base, (uint32_t*)(base + piece)};
  int32_t* val[2] = {(int32_t*)(base + 2 * piece), (int32_t*)(base + 3 * piece)};
  uint32_t* hist0 = (uint32_t*)(base + 4 * piece);
  uint32_t* hist1 = hist0 + (int64_t)rows0 * kSortBins;
  uint32_t* hist2 = hist1 + (int64_t)tiles * kSortBins;
  const int64_t clear = 2 * (int64_t)tiles * kSortBins;
  if (E % 4 == 0) bpr_key_kernel<true><<<dim3((unsigned)rows0), dim3(256), 0, s>>>(logits, T, (int)E, (int)subs, key[0], val[0], hist0, hist1, clear);
  else bpr_key_kernel<false><<<dim3((unsigned)rows0), dim3(256), 0, s>>>(logits, T, (int)E, (int)subs, key[0], val[0], hist0, hist1, clear);
  const dim3 grid((unsigned)tiles), block(1024);
  bpr_sort_kernel<<<grid, block, 0, s>>>(key[0], val[0], T, (int)subs, 0, hist0, rows0, 4, hist1, key[1], val[1]);
  bpr_sort_kernel<<<grid, block, 0, s>>>(key[1], val[1], T, (int)subs, kSortBits, hist1, tiles, 1, hist2, key[0], val[0]);
  bpr_sort_kernel<<<grid, block, 0, s>>>(key[0], val[0], T, (int)subs, 2 * kSortBits, hist2, tiles, 1, nullptr, key[1], val[1]);
  *perm = val[1];
  return hipGetLastError();
}

}  // namespace moe
