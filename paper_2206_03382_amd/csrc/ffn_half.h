// The grouped GEMM of ffn_mfma.hip on half of its large tile: 128 x 256, two blocks to a compute unit, for launches where whole
// tiles of 256 rows divide badly: experts of a few hundred rows, or few tiles per unit.  Included by ffn_mfma.hip (same helpers,
// forward layout, shapes and results: the sums of an output run over k in the same order).
//
// Four waves side by side, each 128 rows x 64 columns as 8 x 4 tiles of v_mfma_f32_16x16x32_bf16 (128 accumulator registers): two
// blocks fit a unit's registers, and one block's matrix instructions run while the other searches its tile, waits for
// its first loads or applies the activation.  K advances by 32 through a three-stage LDS ring (3 x 24 KB) filled by
// direct loads two K-steps ahead.  A wave reads half of its A fragments per half K-step and B's for the next K-step in
// the second half; one barrier per K-step, in its middle, hands the stages over.  All K-steps run through one loop
// body: with the first and last peeled off, the compiler spilled outside the loop and put waits for those reloads inside
// it, which the direct loads then paid for (8 experts x 4096 rows, 2048 x 2048, two products: 650 us, 500 with one body).
//
// What bounds it is the way from L2 into LDS: 24 KB per 128 x 256 x 32 products, half as much again as the large tile, so that
// tile stays the faster where its rounds are full (8 experts x 2048 rows, 2048 x 2048, two products: 239 us there, 268 here), and this one is
// where they are not (8 x 1100: 181 and 165; 32 x 784, 768 x 3072: 327 and 315; numbered in groups throughout).
//
// LDS layouts: A [rows][4 pieces of 8 k], piece g of row r at g ^ (-(r / 4) % 4): the lanes that share a cycle of a
// ds_read_b128 (0-3, 12-15, 20-27 and so on) then cover all 64 banks; with g ^ (r / 4 % 4) two of them meet in every bank.  B
// as in the large tile.
namespace {

constexpr int HBM = kLargeTile / 2, HBN = kLargeTile, HBK = 32, HNS = 3;
constexpr int kHalfA = HBM * HBK * 2, kHalfStage = (HBM + HBN) * HBK * 2;      // 8 KB, 24 KB
constexpr int kHalfLoads = kHalfStage / 4096;                                  // direct loads per wave and K-step

template <int NI>
__device__ __forceinline__ void half_main_loop(char* smem, const char* a_base, const char* b_base, const uint32_t (&a_voff)[2],
                                               const uint32_t (&b_voff)[4], int64_t a_step, int64_t b_step, int a_off,
                                               const int (&b_off)[4], int wave, int KT, const uint16_t* bias_w, int kq, f32x4 (&acc)[8][4]) {
  bf16x8 a[8], b[2][4];
  const uint32_t smem_addr = (uint32_t)(uintptr_t)LDS_PTR(char, smem);
  auto join = [](short4v lo, short4v hi) -> bf16x8 {
    return __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  auto read_a = [&](const char* stage, int i) {
    if (i < 2 * NI) a[i] = *LDS_PTR(bf16x8, stage + a_off + i * 1024);
  };
  auto read_b = [&](const char* stage, int j, bf16x8 (&d)[4]) {
    d[j] = join(__builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4v, stage + b_off[j])),
                __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4v, stage + b_off[j] + 2048)));
  };
  auto mfma = [&](int i, int j, const bf16x8 (&c)[4]) {
    if (i < 2 * NI) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(c[j], a[i], acc[i][j], 0, 0, 0);
  };
  int wstage = 0;                                                   // byte offset of the stage the next loads fill
  const char* a_src = a_base;
  const char* b_src = b_base;
  auto dma = [&](int q) {                                           // load q of the K-step at a_src, b_src
    const uint32_t dst = smem_addr + wstage + wave * 1024;
    if (q < 2) global_to_lds_16(a_src, a_voff[q], dst + q * 4096);
    else global_to_lds_16(b_src, b_voff[q - 2], dst + kHalfA + (q - 2) * 4096);
  };
  auto dma_next = [&]() {
    a_src += a_step;
    b_src += b_step;
    wstage = wstage == 2 * kHalfStage ? 0 : wstage + kHalfStage;
  };
  int rstage = 0;                                                   // stage of the K-step at hand
  auto kstep = [&](int left, bf16x8 (&bc)[4], bf16x8 (&bn)[4]) {    // left: K-steps after this one
    const char* cur = smem + rstage;
    rstage = rstage == 2 * kHalfStage ? 0 : rstage + kHalfStage;
    const char* nxt = smem + rstage;
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      mfma(m >> 2, m & 3, bc);
      PIN();
      if (m < 8 && m % 2 == 0) read_a(cur, 4 + m / 2);
      PIN();
    }
    if (left >= 2) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(kHalfLoads) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    PIN();
    asm volatile("s_barrier" ::: "memory");
    PIN();
    if (left >= 3) {
#pragma unroll
      for (int q = 0; q < kHalfLoads; ++q) dma(q);
      dma_next();
    }
    PIN();
#pragma unroll
    for (int m = 0; m < 16; ++m) {
      mfma(4 + (m >> 2), m & 3, bc);
      PIN();
      if (m == 0) read_a(nxt, 0);
      if (m >= 1 && m < 5) read_b(nxt, m - 1, bn);
      if (m >= 5 && m < 8) read_a(nxt, m - 4);
      PIN();
    }
  };
#pragma unroll
  for (int t = 0; t < HNS; ++t) {
    if (t < KT) {
#pragma unroll
      for (int q = 0; q < kHalfLoads; ++q) dma(q);
    }
    dma_next();
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (bias_w) {
      const u32x2 bb = *reinterpret_cast<const u32x2*>(bias_w + j * 16 + 4 * kq);
      v = f32x4{__uint_as_float(bb.x << 16), __uint_as_float(bb.x & 0xffff0000u), __uint_as_float(bb.y << 16), __uint_as_float(bb.y & 0xffff0000u)};
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) if (i < 2 * NI) acc[i][j] = v;
  }
  PIN();
  if (KT > 2) asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  PIN();
  asm volatile("s_barrier" ::: "memory");
  PIN();
#pragma unroll
  for (int i = 0; i < 4; ++i) read_a(smem, i);
#pragma unroll
  for (int j = 0; j < 4; ++j) read_b(smem, j, b[0]);
  PIN();
#pragma unroll 1
  for (int left = KT - 1; left > 0; left -= 2) {                    // K-steps come in pairs (KT is even)
    kstep(left, b[0], b[1]);
    kstep(left - 1, b[1], b[0]);
  }
}

}  // namespace

template <int ACT>
__global__ __launch_bounds__(256, 2) void grouped_gemm_half_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ B,
                                                                   const uint16_t* __restrict__ bias, const int32_t* __restrict__ counts,
                                                                   const int32_t* __restrict__ gather, int gather_rows, int E, int64_t C, int K, int N,
                                                                   int MT, int NT, uint16_t* __restrict__ out) {
  __shared__ __attribute__((aligned(1024))) char smem[HNS * kHalfStage];
  const int lane = threadIdx.x & 63;
  int e, mt, nt, rows_e;
  if (!find_tile<HBM, false, kHalfGroupShift, true>(blockIdx.x, lane, E, C, counts, NT, e, mt, nt, rows_e)) return;
  const int64_t rows = rows_e;
  const int64_t m0 = (int64_t)mt * HBM;
  if (m0 >= rows) return;
  const int n0 = nt * HBN;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kq = lane >> 4;
  const char* a_base = gather ? (const char*)A : (const char*)(A + (int64_t)e * C * K);
  const char* b_base = (const char*)(B + (int64_t)e * K * N);
  const int KT = K / HBK;
  uint32_t a_voff[2], b_voff[4];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int r = (q * 4 + wave) * 16 + (lane >> 2);
    const int g = (lane & 3) ^ (-(r >> 2) & 3);
    int64_t row = m0 + r;
    row = row < rows ? row : rows - 1;                              // rows past the fill repeat the last one (never stored)
    if (gather) {
      const int t = gather[(int64_t)e * C + row];
      row = (unsigned)t < (unsigned)gather_rows ? t : 0;
    }
    a_voff[q] = (uint32_t)((row * K + g * 8) * 2);
  }
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int kr = (q * 4 + wave) * 2 + (lane >> 5);
    const int c = (lane & 31) ^ (4 * (kr & 3)) ^ (2 * ((kr >> 3) & 1));
    b_voff[q] = (uint32_t)(((int64_t)kr * N + n0 + c * 8) * 2);
  }
  const int64_t a_step = HBK * 2, b_step = (int64_t)HBK * N * 2;
  // LDS read offsets of this lane's fragments: A's sub-tile 0 (1024 bytes apart), B's four
  const int a_off = (lane & 15) * 64 + ((kq ^ (-((lane & 15) >> 2) & 3)) << 4);
  int b_off[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int kr = (lane & 15) >> 2, c = wave * 8 + 2 * j + ((lane & 3) >> 1);
    b_off[j] = kHalfA + (kq * 8 + kr) * 512 + ((c ^ (4 * kr) ^ (2 * (kq & 1))) << 4) + ((lane & 1) << 3);
  }
  const int64_t live = rows - m0;
  const int ni = live >= HBM ? 4 : (int)((live + 31) >> 5);
  f32x4 acc[8][4];
  const uint16_t* bias_w = bias ? bias + (int64_t)e * N + n0 + wave * 64 : nullptr;
#define MOE_TILE_LOOP(NI) half_main_loop<NI>(smem, a_base, b_base, a_voff, b_voff, a_step, b_step, a_off, b_off, wave, KT, bias_w, kq, acc)
  switch (ni) {
    case 4: MOE_TILE_LOOP(4); break;
    case 3: MOE_TILE_LOOP(3); break;
    case 2: MOE_TILE_LOOP(2); break;
    default: MOE_TILE_LOOP(1); break;
  }
#undef MOE_TILE_LOOP
  // epilogue: after the last barrier no wave reads the stages (but for what the last K-step reads ahead and nobody uses), so wave w
  // takes 16 KB as its own: [128 rows][8 pieces of 8 columns], piece c of row r at c ^ (r % 8); stores of 8 rows x 128 bytes.
  char* wtile = smem + wave * 16384;
  uint16_t* oute = out + ((int64_t)e * C + m0) * N + n0 + wave * 64;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    if (i >= 2 * ni) break;
    const int r = i * 16 + (lane & 15);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      u32x2 pk;
      pk.x = pack_bf16x2(epilogue_act<ACT>(acc[i][j][0]), epilogue_act<ACT>(acc[i][j][1]));
      pk.y = pack_bf16x2(epilogue_act<ACT>(acc[i][j][2]), epilogue_act<ACT>(acc[i][j][3]));
      *LDS_PTR(u32x2, wtile + r * 128 + (((2 * j + (kq >> 1)) ^ (r & 7)) << 4) + 8 * (kq & 1)) = pk;
    }
  }
#pragma unroll 4
  for (int it = 0; it < 4 * ni; ++it) {
    const int r = it * 8 + (lane >> 3);
    const u32x4 q = *LDS_PTR(u32x4, wtile + r * 128 + ((lane & 7) << 4));
    if (r < live) *reinterpret_cast<u32x4*>(oute + (int64_t)r * N + (((lane & 7) ^ (r & 7)) << 3)) = q;
  }
}
