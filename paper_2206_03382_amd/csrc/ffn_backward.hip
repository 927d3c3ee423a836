// Backward of the local experts' feed-forward layer (arXiv 2206.03382 Sec. 3.2: the backward pass runs "the backward
// computation of the expert" between the two all-to-alls):  y = act(z W1 + b1) W2 + b2  per expert, so
//   dH = dY W2^T,  dP = dH * act'(z W1 + b1),  dZ = dP W1^T,  dW1 = Z^T dP,  db1 = colsum dP,  dW2 = hidden^T dY,
//   db2 = colsum dY,  over the rows of an expert that exist.
// Every product runs on the grouped GEMM in the operand layout the chain rule asks for (ffn_mfma.hip): the weights are read
// as stored for the products with W^T, the activations as stored for the weight gradients (reduction over an expert's slots
// up to its fill), and act' is applied in the epilogue of the dH product; nothing is copied, padded or transposed in memory.
#include "common.h"
#include "ffn_rules.h"

namespace moe {

namespace {

__device__ __forceinline__ int64_t live_rows(const int32_t* limit, int e, int64_t R) {
  if (!limit) return R;
  const int64_t c = limit[e];
  return c < R ? (c > 0 ? c : 0) : R;
}

// out[e, c] = sum over the live rows r of src[e, r, c], fp32, in a fixed order: 32 interleaved row classes, each summed
// in ascending row order by one thread (16-byte pieces, NP of them per block), then added in class
// order (NP: 8; 16 where slabs are streamed).  Eight rows
// of a class are in flight at a time.   src [E,C,W] as rows of cpr pieces, out [E,W].  Both bias gradients of the layer go in one launch (blocks below
// first.blocks sum the first matrix): for layers of few tokens the launches are what they cost
// (training step of 3001 tokens 334 -> 329 us, fp32 step of 4096 607 -> 601).
template <typename ET> struct ColsumJob {
  const uint4* src;
  ET* out;
  int cpr, blocks;
};
template <typename ET, int NP, bool STREAM>
__global__ __launch_bounds__(32 * NP) void colsum_kernel(const ColsumJob<ET> first, const ColsumJob<ET> second,
                                                     const int32_t* __restrict__ limit, int64_t C) {
  const bool other = (int)blockIdx.x >= first.blocks;
  const uint4* __restrict__ src = other ? second.src : first.src;
  ET* __restrict__ out = other ? second.out : first.out;
  const int cpr = other ? second.cpr : first.cpr, block = other ? blockIdx.x - first.blocks : blockIdx.x;
  constexpr int N = Vec16<ET>::N;
  __shared__ float part[32][NP * N + 1];
  const int e = blockIdx.y;
  const int rc = threadIdx.x / NP, pc = threadIdx.x % NP;
  const int64_t piece = (int64_t)block * NP + pc;
  const int64_t rows = live_rows(limit, e, C);
  float s[N];
#pragma unroll
  for (int u = 0; u < N; ++u) s[u] = 0.f;
  if (piece < cpr) {
    const uint4* at = src + ((int64_t)e * C + rc) * cpr + piece;
    auto add = [&](const uint4& v) __attribute__((always_inline)) {
      float f[N];
      Vec16<ET>::unpack(v, f);
#pragma unroll
      for (int u = 0; u < N; ++u) s[u] += f[u];
    };
    int64_t r = rc;
    for (; r + 7 * 32 < rows; r += 8 * 32, at += (int64_t)8 * 32 * cpr) {
      uint4 v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) v[i] = STREAM ? load_stream(at + (int64_t)i * 32 * cpr) : at[(int64_t)i * 32 * cpr];
#pragma unroll
      for (int i = 0; i < 8; ++i) add(v[i]);
    }
#pragma unroll 4
    for (; r < rows; r += 32, at += (int64_t)32 * cpr) add(*at);
  }
#pragma unroll
  for (int u = 0; u < N; ++u) part[rc][pc * N + u] = s[u];
  __syncthreads();
  if (threadIdx.x < NP * N) {
    const int64_t col = (int64_t)block * NP * N + threadIdx.x;
    if (col < (int64_t)cpr * N) {
      float t = 0.f;
#pragma unroll
      for (int k = 0; k < 32; ++k) t += part[k][threadIdx.x];
      store_from_f32<ET>(out + (int64_t)e * cpr * N + col, t);
    }
  }
}

inline size_t align256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

FfnBackwardWorkspace ffn_backward_layout(int64_t E, int64_t C, int64_t M, int64_t H, int dtype) {
  const size_t es = dtype == MOE_F32 ? 4 : 2;
  const int64_t W = M > H ? M : H;
  FfnBackwardWorkspace w;
  size_t o = 0;
  w.pre = o;  o += align256((size_t)E * C * H * es);
  w.dP = o;   o += align256((size_t)E * C * H * es);
  w.a_tail = o;  o += align256(grouped_gemm_tn_tail_bytes(E, W));
  w.b_tail = o;  o += align256(grouped_gemm_tn_tail_bytes(E, W));
  w.total = o;
  return w;
}

template <typename ET>
static hipError_t ffn_backward_t(const void* Z, const void* W1, const void* b1, const void* W2, const void* saved_pre,
                                 const void* hidden, const void* dY, int act, int dtype, const int32_t* counts, int64_t E, int64_t C, int64_t M,
                                 int64_t H, char* ws, void* dZ, void* dW1, void* db1, void* dW2, void* db2, hipStream_t s,
                                 int64_t rows_hint, const int32_t* gather, int64_t gather_rows) {
  const FfnBackwardWorkspace w = ffn_backward_layout(E, C, M, H, dtype);
  const int es = (int)sizeof(ET);
  void *dP = ws + w.dP, *a_tail = ws + w.a_tail, *b_tail = ws + w.b_tail;
  const void* pre = saved_pre ? saved_pre : ws + w.pre;
  hipError_t err;
#define MOE_TRY(x) do { err = (x); if (err != hipSuccess) return err; } while (0)
  // pre-activations: the caller's (kept by the training forward), else recomputed
  if (!saved_pre) {
    if (gather) return hipErrorInvalidValue;                       // a fused-dispatch training forward always keeps them
    MOE_TRY(launch_grouped_gemm(Z, W1, b1, -1, dtype, counts, E, C, M, H, ws + w.pre, s, rows_hint));
  }
  auto colsums = [&]() -> hipError_t {
    const int cprH = (int)(H * es / 16), cprM = (int)(M * es / 16);
    const bool stream = colsum_streams(E, counts ? mean_or(rows_hint, C) : (double)C, db1 ? H * es : 0, db2 ? M * es : 0);
    const int np = stream ? 16 : 8;
    const ColsumJob<ET> j1 = {(const uint4*)dP, (ET*)db1, cprH, db1 ? (int)ceil_div(cprH, np) : 0};
    const ColsumJob<ET> j2 = {(const uint4*)dY, (ET*)db2, cprM, db2 ? (int)ceil_div(cprM, np) : 0};
    if (j1.blocks + j2.blocks == 0) return hipSuccess;
    const dim3 grid((unsigned)(j1.blocks + j2.blocks), (unsigned)E);
    if (stream) colsum_kernel<ET, 16, true><<<grid, dim3(512), 0, s>>>(j1, j2, counts, C);
    else colsum_kernel<ET, 8, false><<<grid, dim3(256), 0, s>>>(j1, j2, counts, C);
    return hipGetLastError();
  };
  // dP = (dY W2^T) * act'(pre);  dZ = dP W1^T;  dW2 = hidden^T dY;  dW1 = Z^T dP
  MOE_TRY(launch_grouped_gemm_nt(dY, W2, dtype, counts, E, C, M, H, dP, pre, act, s, rows_hint));
  if (dZ) MOE_TRY(launch_grouped_gemm_nt(dP, W1, dtype, counts, E, C, H, M, dZ, nullptr, -1, s, rows_hint));
  if (dW2) MOE_TRY(launch_grouped_gemm_tn(hidden, dY, dtype, counts, E, C, H, M, a_tail, b_tail, dW2, s, rows_hint));
  if (dW1) MOE_TRY(launch_grouped_gemm_tn(Z, dP, dtype, counts, E, C, M, H, a_tail, b_tail, dW1, s, rows_hint, gather, gather_rows));
  MOE_TRY(colsums());
#undef MOE_TRY
  return hipSuccess;
}

hipError_t launch_expert_ffn_backward(const void* Z, const void* W1, const void* b1, const void* W2, const void* pre,
                                      const void* hidden, const void* dY, int act, int dtype, const int32_t* counts, int64_t E,
                                      int64_t C, int64_t M, int64_t H, void* ws, void* dZ, void* dW1, void* db1, void* dW2,
                                      void* db2, hipStream_t s, int64_t rows_hint, const int32_t* gather, int64_t gather_rows) {
  if (dtype == MOE_F32)
    return ffn_backward_t<float>(Z, W1, b1, W2, pre, hidden, dY, act, dtype, counts, E, C, M, H, (char*)ws, dZ, dW1, db1, dW2, db2, s,
                                 rows_hint, gather, gather_rows);
  return ffn_backward_t<uint16_t>(Z, W1, b1, W2, pre, hidden, dY, act, dtype, counts, E, C, M, H, (char*)ws, dZ, dW1, db1, dW2, db2, s,
                                  rows_hint, gather, gather_rows);
}

}  // namespace moe
