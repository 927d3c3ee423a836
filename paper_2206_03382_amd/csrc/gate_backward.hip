// Backward of the gating function (arXiv 2206.03382 Sec. 2.1 gate; Sec. 3.2: the backward pass mirrors the forward).
//   gate_backward_kernel : d gate_w [T,k] -> d logits [T,E] through (renormalised) softmax-at-the-chosen-experts, and the
//                          operands of the two products below
//   gate_dx_kernel       : dx[t,:] = sum_e dlogits[t,e] Wg[:,e] + what the dispatch's backward brings, for narrow gates
//                          (wide ones: a product on the grouped GEMM)
//   dWg[m,e] = sum_t x[t,m] dlogits[t,e]: token slices on the grouped GEMM's kernels
//   gate_dw_reduce_kernel: sums of the token slices of dWg, and of the token blocks of dbias, in a fixed order
// The chosen experts and the slots are integer decisions and carry no gradient.
//
// dlogits stay fp32 in dWg of a bf16 gate: a value is the exact sum of three bf16 values (each the round-to-nearest of what is
// left), and a product with it the sum of three matrix-core products with those.  The three make 3 Ep columns [T, 3 Ep] (Ep = E
// padded to 8) that share every read of x.  Infinities: the second and third pieces of a value that is not finite are 0, and a
// sum over first pieces that is not finite stands for the whole, so an infinite token entry gives what the plain product gives.
#include "common.h"
#include "gate_rules.h"

namespace moe {

namespace {

// G lanes per token (8, 16, or 64 for gates of more than 128 experts), lane gl holds experts gl + G i.  p = softmax(logits);
// g_j = p[idx_j]; gate_w = g / sum g (normalize) or g.  A block walks `rounds` rounds of 256 / G tokens; with `pbias` it adds up
// their dlogits per expert, in token order, through LDS.  dl [T,E] fp32 (optional); dcols: [T, 3 Ep] bf16 pieces or, SPLIT
// false, [T, Ep] fp32 (optional); dl16 [T, E64] bf16, zero-padded (optional).  All blocks
// together write wgp [M, Ep], Wg with zero-padded rows (optional; blocks past the last token do only that, so that few tokens
// do not leave it to one or two: dx of 64 tokens, bf16, M = 4096, 4 experts 16.0 -> 9.3 us).
// Bound by its loads' latency.  One thread per token, which this replaced, was a serial chain of 3 E exponentials: 65536 tokens,
// 128 experts 62 us, now 27; 8 experts 8.5, now 6.2.
struct GateBackwardArgs {
  const float* logits;
  const int32_t* idx;
  const float* dgate_w;
  int64_t T;
  int E, k, normalize, Ep, E64, rounds;
  float* dl;
  void* dcols;
  uint16_t* dl16;
  float* pbias;
  const uint16_t* Wg;
  uint16_t* wgp;
  int64_t M;
};

template <int G, int V, bool SPLIT>
__global__ __launch_bounds__(256) void gate_backward_kernel(const GateBackwardArgs a) {
  extern __shared__ float rows[];                           // [tokens of the block][E + 1], with pbias
  constexpr int TOK = 256 / G;
  const int g = threadIdx.x / G, gl = threadIdx.x % G;
  if (a.wgp) {
    const int64_t n = a.M * a.Ep;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
      const int e = (int)(i % a.Ep);
      a.wgp[i] = e < a.E ? a.Wg[i / a.Ep * a.E + e] : (uint16_t)0;
    }
  }
  if ((int64_t)blockIdx.x * (TOK * a.rounds) >= a.T) return;
  auto sum = [](float v) {
#pragma unroll
    for (int d = 1; d < G; d <<= 1) v += __shfl_xor(v, d, 64);
    return v;
  };
  for (int rd = 0; rd < a.rounds; ++rd) {
    const int tb = rd * TOK + g;
    const int64_t t = (int64_t)blockIdx.x * (TOK * a.rounds) + tb;
    const bool valid = t < a.T;                             // the same in all lanes of a group
    float p[V], dw[V], dl[V];
    bool chosen[V];
    float mx = -__builtin_inff();
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int e = gl + G * i;
      p[i] = valid && e < a.E ? a.logits[t * a.E + e] : -__builtin_inff();
      chosen[i] = false;
      dw[i] = 0.f;
      mx = fmaxf(mx, p[i]);
    }
#pragma unroll
    for (int d = 1; d < G; d <<= 1) mx = fmaxf(mx, __shfl_xor(mx, d, 64));
    float se = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int e = gl + G * i;
      p[i] = e < a.E ? expf(p[i] - mx) : 0.f;
      se += p[i];
    }
    const float inv = 1.0f / sum(se);
#pragma unroll
    for (int i = 0; i < V; ++i) p[i] *= inv;
    if (valid) {
      for (int j = 0; j < a.k; ++j) {                       // the chosen experts of a token are distinct
        const int e = a.idx[t * a.k + j];
        const float d = a.dgate_w[t * a.k + j];
#pragma unroll
        for (int i = 0; i < V; ++i)
          if (e == gl + G * i && e < a.E) { chosen[i] = true; dw[i] = d; }
      }
    }
    float S = 1.f, c1 = 0.f;
    if (a.normalize) {
      float s = 0.f;
#pragma unroll
      for (int i = 0; i < V; ++i) s += chosen[i] ? p[i] : 0.f;
      S = sum(s);
      s = 0.f;
#pragma unroll
      for (int i = 0; i < V; ++i) s += chosen[i] ? dw[i] * (p[i] / S) : 0.f;
      c1 = sum(s);
    }
    // dg_j = (dw_j - c1) / S;   c = sum_j g_j dg_j = sum_e p_e dp_e
    float c = 0.f;
#pragma unroll
    for (int i = 0; i < V; ++i) c += chosen[i] ? p[i] * ((dw[i] - c1) / S) : 0.f;
    c = sum(c);
#pragma unroll
    for (int i = 0; i < V; ++i) dl[i] = -p[i] * c + (chosen[i] ? p[i] * ((dw[i] - c1) / S) : 0.f);
    if (!valid) continue;
#pragma unroll
    for (int i = 0; i < V; ++i) {
      const int e = gl + G * i;
      const float v = e < a.E ? dl[i] : 0.f;
      if (a.dl && e < a.E) a.dl[t * a.E + e] = v;
      if (a.dl16 && e < a.E64) a.dl16[t * a.E64 + e] = f32_to_bf16_bits(v);
      if (a.dcols && e < a.Ep) {
        if (SPLIT) {
          uint16_t* d = (uint16_t*)a.dcols + t * 3 * a.Ep + e;
          float left = v;
#pragma unroll
          for (int q = 0; q < 3; ++q) {
            const uint16_t b = f32_to_bf16_bits(left);
            d[q * a.Ep] = b;
            const float r = left - bf16_bits_to_f32(b);
            left = (b & 0x7f80) == 0x7f80 ? 0.f : r;
          }
        } else {
          ((float*)a.dcols)[t * a.Ep + e] = v;
        }
      }
      if (a.pbias && e < a.E) rows[tb * (a.E + 1) + e] = v;
    }
    if (a.dl16)
      for (int e = gl + G * V; e < a.E64; e += G) a.dl16[t * a.E64 + e] = 0;
  }
  if (a.pbias) {
    __syncthreads();
    const int64_t t0 = (int64_t)blockIdx.x * (TOK * a.rounds);
    const int n = (int)(a.T - t0 < TOK * a.rounds ? a.T - t0 : TOK * a.rounds);
    for (int e = threadIdx.x; e < a.E; e += 256) {
      float s = 0.f;
#pragma unroll 8
      for (int tt = 0; tt < n; ++tt) s += rows[tt * (a.E + 1) + e];
      a.pbias[(int64_t)blockIdx.x * a.E + e] = s;
    }
  }
}

// Eight consecutive entries of row `row` of a matrix [., ld] starting at column e0, as floats (0 past E).  With `vec` (ld a
// multiple of 8, 16-byte aligned) the pieces are fetched whole.
template <typename ET>
__device__ __forceinline__ void wg_row8(const ET* __restrict__ Wg, int64_t row, int ld, int E, int e0, bool vec, float (&out)[8]) {
  constexpr int N = Vec16<ET>::N;
  if (vec) {
    const uint4* p = reinterpret_cast<const uint4*>(Wg + row * ld + e0);
#pragma unroll
    for (int h = 0; h < 8 / N; ++h) {
      float f[N];
      Vec16<ET>::unpack(p[h], f);
#pragma unroll
      for (int i = 0; i < N; ++i) out[h * N + i] = f[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) out[i] = e0 + i < E ? load_as_f32<ET>(Wg + row * ld + e0 + i) : 0.f;
  }
}

// dx[t,m] = before + sum_e dlogits[t,e] Wg[m,e], summed in fp32.  before: 0, dx itself (accumulate), or, with `slabs` [E,C,M], the
// sum of the token's kept slot rows in rank order, rounded to the storage type (the dispatch's backward, bit for bit, which
// then needs no pass over dx of its own).  A
// thread owns one 16-byte piece of the rows (N consecutive m) for TT tokens: all their pieces are in flight at once and
// stay in registers while its N rows of Wg pass by, 8 experts at a time; the block's dlogits go through LDS.  Bound by the
// slabs' and dx's bytes: 16384 tokens, M = 2048, 8 experts, top-2: 49 us (4.1 TB/s), for what took 39 + 33 us in two passes.
// Few tokens take blocks of 4, to spread over the chip (3001 tokens, M = 776, 17 experts: 13 us instead of 5 + 27).
constexpr int kDxMaxChoices = 32;
template <typename ET, int TT>
__global__ __launch_bounds__(256) void gate_dx_kernel(const float* __restrict__ dlogits, const ET* __restrict__ Wg, int ldw, int64_t T,
                                                      int cpr, int E, int accumulate, const uint4* __restrict__ slabs,
                                                      const int32_t* __restrict__ idx, const int32_t* __restrict__ loc, int k,
                                                      int64_t C, uint4* __restrict__ dx) {
  constexpr int N = Vec16<ET>::N;
  __shared__ float dls[TT][8];
  __shared__ int64_t rows[kDxMaxChoices][TT];               // slab row of choice j of token tt, -1: dropped
  const int64_t t0 = (int64_t)blockIdx.x * TT;
  const int piece = blockIdx.y * blockDim.x + threadIdx.x;
  const bool live = piece < cpr;                            // every thread joins the barriers
  const bool vec = (ldw % 8) == 0 && (reinterpret_cast<uintptr_t>(Wg) & 15) == 0;
  float acc[TT][N];
#pragma unroll
  for (int tt = 0; tt < TT; ++tt) {
    if (live && accumulate && t0 + tt < T) Vec16<ET>::unpack(dx[(t0 + tt) * cpr + piece], acc[tt]);
    else {
#pragma unroll
      for (int u = 0; u < N; ++u) acc[tt][u] = 0.f;
    }
  }
  if (slabs) {
    for (int i = threadIdx.x; i < k * TT; i += blockDim.x) {
      const int64_t t = t0 + i / k;
      int64_t row = -1;
      if (t < T) {
        const int e = idx[t * k + i % k], l = loc[t * k + i % k];
        if (l >= 0 && l < C && (unsigned)e < (unsigned)E) row = (int64_t)e * C + l;
      }
      rows[i % k][i / k] = row;
    }
    __syncthreads();
    for (int j = 0; j < k; ++j) {
      uint4 v[TT];
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) v[tt] = live && rows[j][tt] >= 0 ? slabs[rows[j][tt] * cpr + piece] : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
        float f[N];
        Vec16<ET>::unpack(v[tt], f);
#pragma unroll
        for (int u = 0; u < N; ++u) acc[tt][u] += f[u];
      }
    }
#pragma unroll
    for (int tt = 0; tt < TT; ++tt) Vec16<ET>::unpack(Vec16<ET>::pack(acc[tt]), acc[tt]);
  }
  for (int e0 = 0; e0 < E; e0 += 8) {
    __syncthreads();                                        // the previous chunk's dlogits have been read
    for (int i = threadIdx.x; i < TT * 8; i += blockDim.x) {
      const int tt = i >> 3, u = i & 7;
      dls[tt][u] = (t0 + tt < T && e0 + u < E) ? dlogits[(t0 + tt) * E + e0 + u] : 0.f;
    }
    __syncthreads();
    if (live) {
      float wr[N][8];
#pragma unroll
      for (int u = 0; u < N; ++u) wg_row8<ET>(Wg, (int64_t)piece * N + u, ldw, E, e0, vec, wr[u]);
#pragma unroll
      for (int tt = 0; tt < TT; ++tt) {
#pragma unroll
        for (int u = 0; u < N; ++u)
#pragma unroll
          for (int i = 0; i < 8; ++i) acc[tt][u] = fmaf(dls[tt][i], wr[u][i], acc[tt][u]);
      }
    }
  }
  if (live) {
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
      if (t0 + tt < T) dx[(t0 + tt) * cpr + piece] = Vec16<ET>::pack(acc[tt]);
  }
}

// dWg[m, e] = sum over the slices, in order, of part[s][m][e] (+ the second and third pieces' sums, unless the first is not
// finite); dbias[e] = sum over the token blocks, in order, of pbias[b][e].  A block owns 32 results, eight threads each: a
// thread adds a contiguous eighth of the slices, the eighths are added in order.
template <typename ET>
__global__ __launch_bounds__(256) void gate_dw_reduce_kernel(const float* __restrict__ part, int64_t M, int E, int Ep, int pieces,
                                                             int slices, ET* __restrict__ dWg, int64_t dw_blocks,
                                                             const float* __restrict__ pbias, int nb, float* __restrict__ dbias) {
  __shared__ float sums[8][3][33];
  const int r = threadIdx.x & 31, g = threadIdx.x >> 5;
  const bool bias = blockIdx.x >= dw_blocks;
  const int64_t i = (bias ? blockIdx.x - dw_blocks : (int64_t)blockIdx.x) * 32 + r;
  const int64_t n = bias ? E : M * E;
  const int count = bias ? nb : slices, np = bias ? 1 : pieces, per = (count + 7) / 8;
  const int s0 = g * per, s1 = s0 + per < count ? s0 + per : count;
  const int64_t row = bias ? E : M * pieces * Ep;           // floats per slice
  const float* src = bias ? pbias + i : part + (i / E) * pieces * Ep + i % E;
  for (int q = 0; q < np; ++q) {
    float s = 0.f;
    if (i < n) {
#pragma unroll 8
      for (int k = s0; k < s1; ++k) s += src[k * row + q * Ep];
    }
    sums[g][q][r] = s;
  }
  __syncthreads();
  if (g > 0 || i >= n) return;
  float t[3] = {0.f, 0.f, 0.f};
  for (int q = 0; q < np; ++q)
#pragma unroll
    for (int h = 0; h < 8; ++h) t[q] += sums[h][q][r];
  const float v = t[0] - t[0] == 0.f ? t[0] + (t[1] + t[2]) : t[0];
  if (bias) dbias[i] = v;
  else store_from_f32<ET>(dWg + i, v);
}

// The workspace: dlogits, partial sums of dbias and dWg, the products' operands (each only where it is needed)
struct GateBackwardLayout {
  size_t dl, pbias, part, dcols, wgp, dl16, total;
  int64_t Ep, E64;
};

GateBackwardLayout gate_backward_layout(int64_t T, int64_t M, int64_t E) {
  GateBackwardLayout w;
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t at = off; off = align_up(off + bytes, 256); return at; };
  w.Ep = align_up(E, 8);
  w.E64 = align_up(E, 64);
  auto part_bytes = [&](int dtype, int64_t N) { return (size_t)(gemm_slices(dtype, T, M, N).count * M * N * 4); };
  const size_t bf16 = part_bytes(MOE_BF16, 3 * w.Ep), fp32 = part_bytes(MOE_F32, w.Ep);
  w.dl = take((size_t)T * E * 4);
  w.pbias = take((size_t)ceil_div(T, gate_backward_token_block(T, E, true)) * E * 4);
  w.part = take(bf16 > fp32 ? bf16 : fp32);
  w.dcols = take((size_t)T * 3 * w.Ep * 2);                 // 6 bytes per padded entry, or 4 as fp32
  w.wgp = take((size_t)M * w.Ep * 2);
  w.dl16 = take((size_t)T * w.E64 * 2 + (size_t)M * w.E64 * 2);
  w.total = off;
  return w;
}

// dst [rows, Ep] bf16 = src [rows, E] (fp32 or bf16) with the columns E .. Ep-1 zero; Ep a multiple of 8.  One thread
// per 8 output columns.  Operands of the matrix-core product below (its reduction runs in steps of 64 experts).
template <typename ST>
__global__ __launch_bounds__(256) void pad_to_bf16_kernel(const ST* __restrict__ src, int64_t rows, int E, int Ep,
                                                          uint4* __restrict__ dst) {
  const int gpr = Ep / 8;
  const int64_t n = rows * gpr;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int64_t r = i / gpr;
    const int e0 = (int)(i % gpr) * 8;
    float f[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) f[u] = e0 + u < E ? load_as_f32<ST>(src + r * E + e0 + u) : 0.f;
    dst[i] = Vec16<uint16_t>::pack(f);
  }
}

}  // namespace

// Whether dx is a [T, E] x [E, M] product on the large matrix-core tile, which rounds dlogits to bf16: bf16 gates of 32 experts
// and more.  gate_dx_kernel takes all others, with dlogits in fp32.
static bool wide_dx(int dtype, const void* Wg, int64_t T, int64_t M, int64_t E) {
  const int64_t E64 = align_up(E, 64);
  return dtype == MOE_BF16 && E >= 32 && M % 256 == 0 && (reinterpret_cast<uintptr_t>(Wg) & 15) == 0 && T * E64 < ((int64_t)1 << 31) &&
         M * E64 < ((int64_t)1 << 31);
}

bool gate_backward_takes_slabs(int dtype, const void* Wg, int64_t T, int64_t M, int64_t E, int k) {
  return !wide_dx(dtype, Wg, T, M, E) && k <= kDxMaxChoices;
}

size_t gate_backward_workspace_bytes(int64_t T, int64_t M, int64_t E) { return gate_backward_layout(T, M, E).total; }

template <typename ET>
static hipError_t gate_backward_t(const void* x, const void* Wg, const float* logits, const int32_t* idx, const float* dgate_w,
                                  int normalize, int64_t T, int64_t M, int64_t E, int k, char* ws, void* dx, int accumulate_dx,
                                  void* dWg, float* dbias, float* dlogits_out, hipStream_t s, const void* slabs, const int32_t* loc,
                                  int64_t C) {
  constexpr bool BF16 = sizeof(ET) == 2;
  constexpr int dtype = BF16 ? MOE_BF16 : MOE_F32, pieces = BF16 ? 3 : 1;
  const GateBackwardLayout w = gate_backward_layout(T, M, E);
  // wide dx: Wg [M, E] is the transposed operand as stored, dlogits are rounded to bf16, the reduction runs in steps of 64
  // experts (other counts get zero-padded operands); the accumulate form adds dx in the epilogue
  const bool dx_wide = dx && wide_dx(dtype, Wg, T, M, E);
  const bool pad_wg = BF16 && dx && !dx_wide && E % 8 != 0;
  const int64_t token_block = gate_backward_token_block(T, E, dbias != nullptr);
  GateBackwardArgs a = {logits, idx, dgate_w, T, (int)E, k, normalize, (int)w.Ep, (int)w.E64, (int)(token_block * gate_backward_lanes(E) / 256), dlogits_out, nullptr, nullptr, nullptr,
                        (const uint16_t*)Wg, nullptr, M};
  if (dx && !dx_wide && !a.dl) a.dl = (float*)(ws + w.dl);
  if (dWg) a.dcols = ws + w.dcols;
  if (dx_wide) a.dl16 = (uint16_t*)(ws + w.dl16);
  if (pad_wg) a.wgp = (uint16_t*)(ws + w.wgp);
  if (dbias) a.pbias = (float*)(ws + w.pbias);
  const int nb = (int)ceil_div(T, token_block);
  const int64_t pad_blocks = pad_wg ? ceil_div(M * w.Ep, 256 * 4) : 0;
  const unsigned blocks = (unsigned)(nb >= 256 || pad_blocks <= nb ? nb : (pad_blocks < 256 ? pad_blocks : 256));
  const size_t shmem = dbias ? (size_t)token_block * (E + 1) * sizeof(float) : 0;         // at most 33 KB where memory holds the tokens
#define MOE_GATE_BACKWARD(G, V) gate_backward_kernel<G, V, BF16><<<dim3(blocks), dim3(256), shmem, s>>>(a)
  if (E <= 8) MOE_GATE_BACKWARD(8, 1); else if (E <= 16) MOE_GATE_BACKWARD(16, 1); else if (E <= 32) MOE_GATE_BACKWARD(16, 2); else if (E <= 64) MOE_GATE_BACKWARD(16, 4);
  else if (E <= 128) MOE_GATE_BACKWARD(16, 8); else if (E <= 256) MOE_GATE_BACKWARD(64, 4); else MOE_GATE_BACKWARD(64, 8);
#undef MOE_GATE_BACKWARD
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (dx_wide) {
    const void* wgt = Wg;
    if (w.E64 != E) {
      uint16_t* wg16 = a.dl16 + T * w.E64;
      const int64_t b = ceil_div(M * w.E64 / 8, 256 * 4);
      pad_to_bf16_kernel<uint16_t><<<dim3((unsigned)(b < 8192 ? b : 8192)), dim3(256), 0, s>>>((const uint16_t*)Wg, M, (int)E, (int)w.E64, (uint4*)wg16);
      if ((err = hipGetLastError()) != hipSuccess) return err;
      wgt = wg16;
    }
    err = launch_grouped_gemm_nt(a.dl16, wgt, MOE_BF16, nullptr, 1, T, w.E64, M, dx, accumulate_dx ? dx : nullptr, -1, s);
  } else if (dx) {
    const int cpr = (int)(M * sizeof(ET) / 16);
    const int threads = cpr >= 256 ? 256 : (int)align_up(cpr, 64);
    const unsigned ny = (unsigned)ceil_div(cpr, threads);
    const ET* wg = pad_wg ? (const ET*)a.wgp : (const ET*)Wg;
    const int ldw = pad_wg ? (int)w.Ep : (int)E;
#define MOE_GATE_DX(TT) gate_dx_kernel<ET, TT><<<dim3((unsigned)ceil_div(T, TT), ny), dim3(threads), 0, s>>>(a.dl, wg, ldw, T, cpr, (int)E, accumulate_dx, (const uint4*)slabs, idx, loc, k, C, (uint4*)dx)
    if (gate_dx_tokens(T, M * (int64_t)sizeof(ET)) == 16) MOE_GATE_DX(16); else MOE_GATE_DX(4);
#undef MOE_GATE_DX
    err = hipGetLastError();
  }
  if (err != hipSuccess) return err;
  if (dWg) {
    err = launch_gemm_tn_slices(x, a.dcols, dtype, T, M, pieces * w.Ep, (float*)(ws + w.part), s);
    if (err != hipSuccess) return err;
  }
  if (dWg || dbias) {
    const int64_t dw_blocks = dWg ? ceil_div(M * E, 32) : 0, blocks = dw_blocks + (dbias ? ceil_div(E, 32) : 0);
    const int slices = (int)gemm_slices(dtype, T, M, pieces * w.Ep).count;
    gate_dw_reduce_kernel<ET><<<dim3((unsigned)blocks), dim3(256), 0, s>>>((const float*)(ws + w.part), M, (int)E, (int)w.Ep, pieces, slices,
                                                                           (ET*)dWg, dw_blocks, a.pbias, nb, dbias);
    err = hipGetLastError();
  }
  return err;
}

hipError_t launch_gate_backward(const void* x, const void* Wg, const float* logits, const int32_t* idx, const float* dgate_w,
                                int normalize, int dtype, int64_t T, int64_t M, int64_t E, int k, void* ws, void* dx,
                                int accumulate_dx, void* dWg, float* dbias, float* dlogits, hipStream_t s, const void* slabs,
                                const int32_t* loc, int64_t C) {
  if (slabs && (accumulate_dx || !gate_backward_takes_slabs(dtype, Wg, T, M, E, k))) return hipErrorInvalidValue;
  if (dtype == MOE_F32)
    return gate_backward_t<float>(x, Wg, logits, idx, dgate_w, normalize, T, M, E, k, (char*)ws, dx, accumulate_dx, dWg, dbias, dlogits, s, slabs, loc, C);
  return gate_backward_t<uint16_t>(x, Wg, logits, idx, dgate_w, normalize, T, M, E, k, (char*)ws, dx, accumulate_dx, dWg, dbias, dlogits, s, slabs, loc, C);
}

}  // namespace moe
