// A part of TM x TN of one of the large tile's last tiles (ffn_rules.h: cut_tile).  Included by ffn_mfma.hip; same shapes and results: the sums of
// an output run over k in the same order.
//
// A whole tile has its unit for itself and hides the way from memory behind its own products.  A part has half or a quarter of those, so what it
// waits for is that way, and what hides it is depth: all of the unit's LDS holds NS K-steps of the part, and the loads of K-step kt + NS go out as soon as
// the last read of K-step kt frees its stage.  Four waves of TM/2 x TN/2 as tiles of v_mfma_f32_16x16x32_bf16, one barrier per K-step of 64.  K = 2048: a
// quarter (128 x 128, five K-steps) alone on its XCD takes 13 us, 25 where all units load one, at 50 KB per us and unit; a half (256 x 128, three)
// 36; a whole tile 57.
//
// LDS layouts: a k-contiguous operand as in the large tile, B with k slow as in ffn_ring.h.
namespace {

struct Piece {
  const uint16_t* A;            // the expert's slab, or the gathered matrix
  const uint16_t* B;            // the expert's matrix
  const uint16_t* bias;         // at its columns, or null
  const int32_t* gather;        // slot -> row of A at its rows, or null
  int gather_rows;
  int64_t m0;                   // first row
  int rows;                     // rows from there on that exist, at least one, at most TM
  int n0, K, N;
  int64_t out;                  // offset of its first output
};

// NA: 32-row groups of A that are loaded; NI: 16-row tiles of this wave that are computed.
template <int TM, int TN, int NS, int MODE, int NA, int NI>
__device__ __forceinline__ void piece_main_loop(char* smem, const Piece& p, int lane, int wave, f32x4 (&acc)[TM / 32][TN / 32]) {
  constexpr bool TRB = MODE == kNN;
  constexpr int RA = TM / 32, RB = TN / 32, LB = TN / 32, L = NA + LB;          // 16 x 16 tiles of a wave; direct loads per wave and K-step
  constexpr int A_STAGE = TM * 128, STAGE = A_STAGE + TN * 128;
  constexpr int NM = RA * RB, NR = RA + (TRB ? 2 * RB : RB), SPAN = NM * 3 / 4, BAR = NM * 7 / 8;
  const int wm = wave >> 1, wn = wave & 1, kq = lane >> 4, KT = p.K / kLargeK;
  auto swz_slow = [](int kr) -> int { return (4 * (kr & 3)) ^ (2 * ((kr >> 3) & 1)); };
  const int fast_k = ((lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7)) * 8;

  const char* a_ptr[NA];
  uint32_t b_voff[LB];
#pragma unroll
  for (int q = 0; q < NA; ++q) {
    int r = (q * 4 + wave) * 8 + (lane >> 3);
    r = r < p.rows ? r : p.rows - 1;                                // rows past the fill repeat the last one (never stored)
    int64_t row = p.m0 + r;
    if (p.gather) {
      const int t = p.gather[r];
      row = (unsigned)t < (unsigned)p.gather_rows ? t : 0;
    }
    a_ptr[q] = (const char*)(p.A + row * p.K + fast_k);
  }
#pragma unroll
  for (int q = 0; q < LB; ++q) {
    const int at = (q * 4 + wave) * 64 + lane, kr = at / (TN / 8);
    if (TRB) b_voff[q] = (uint32_t)(((int64_t)kr * p.N + p.n0 + ((at % (TN / 8)) ^ swz_slow(kr)) * 8) * 2);
    else b_voff[q] = (uint32_t)(((int64_t)(p.n0 + (q * 4 + wave) * 8 + (lane >> 3)) * p.K + fast_k) * 2);
  }
  // accumulators: the bias (register u of tile (i, j) is column 16 j + 4 kq + u of the wave's), or zero
#pragma unroll
  for (int j = 0; j < RB; ++j) {
    f32x4 b = {0.f, 0.f, 0.f, 0.f};
    if (MODE == kNN && p.bias) {
      const u32x2 v = *reinterpret_cast<const u32x2*>(p.bias + wn * (TN / 2) + j * 16 + 4 * kq);
      b = f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) acc[i][j] = b;
  }
  PIN();
  const char* b_src = (const char*)p.B;
  const int64_t b_step = TRB ? (int64_t)kLargeK * p.N * 2 : kLargeK * 2;
  const uint32_t smem_addr = (uint32_t)(uintptr_t)LDS_PTR(char, smem);
  auto dma = [&](int n, int stage) __attribute__((always_inline)) {             // load n of a K-step, stage: byte offset
    const uint32_t dst = smem_addr + stage + wave * 1024;
    if (n < NA) {
      global_to_lds_16(a_ptr[n], dst + n * 4096);
      a_ptr[n] += kLargeK * 2;
    } else {
      global_to_lds_16(b_src, b_voff[n - NA], dst + A_STAGE + (n - NA) * 4096);
    }
  };
  // until at most `later` K-steps' loads are in flight (loads return in order)
  auto wait_loads = [&](int later) __attribute__((always_inline)) {
    if (later >= NS - 1) asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NS - 1) * L) : "memory");
    else if (NS > 4 && later == 3) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(3 * L) : "memory");
    else if (NS > 3 && later == 2) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(2 * L) : "memory");
    else if (later == 1) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(L) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  auto read_fast = [&](const char* at, int w, int t, int s) __attribute__((always_inline)) -> bf16x8 {
    return *LDS_PTR(bf16x8, at + (w + t * 16 + (lane & 15)) * 128 + (((4 * s + kq) ^ ((lane & 15) >> 1)) << 4));
  };
  auto read_slow = [&](const char* at, int w, int t, int s, int half) __attribute__((always_inline)) -> short4v {
    const int kr = kq * 8 + ((lane & 15) >> 2), c = w / 8 + 2 * t + ((lane & 3) >> 1);
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        LDS_PTR(short4v, at + kr * TN * 2 + ((c ^ swz_slow(kr)) << 4) + ((lane & 1) << 3) + (32 * s + 4 * half) * TN * 2));
  };
  bf16x8 fa[2][RA], fb[2][RB];
  short4v lo;
  // read number r of sub-step s of the stage at `at` into fragment buffer d: the first of A, B's, then the rest of A's
  auto read = [&](const char* at, int s, int r, int d) __attribute__((always_inline)) {
    if (NI == 0) return;
    if (r >= 1 && r < 1 + NR - RA) {
      const int rb = r - 1;
      if (!TRB) fb[d][rb] = read_fast(at + A_STAGE, wn * (TN / 2), rb, s);
      else if ((rb & 1) == 0) lo = read_slow(at + A_STAGE, wn * (TN / 2), rb >> 1, s, 0);
      else fb[d][rb >> 1] = __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(lo, read_slow(at + A_STAGE, wn * (TN / 2), rb >> 1, s, 1), 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      const int ra = r < 1 ? 0 : r - (NR - RA);
      if (ra < NI) fa[d][ra] = read_fast(at, wm * (TM / 2), ra, s);
    }
  };
  auto mfma = [&](int m, int d) __attribute__((always_inline)) {
    const int i = m / RB, j = m % RB;
    if (i < NI) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[d][j], fa[d][i], acc[i][j], 0, 0, 0);
  };
  int stage = 0;                                                    // byte offset of K-step kt's stage
  auto kstep = [&](auto dma_tag, int kt) __attribute__((always_inline)) {
    constexpr bool DMA = decltype(dma_tag)::value;                  // K-step kt + NS exists
    const char* cur = smem + stage;
    const int fill = stage;
    stage = stage == (NS - 1) * STAGE ? 0 : stage + STAGE;
    const char* nxt = smem + stage;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      mfma(m, 0);
      PIN();
#pragma unroll
      for (int r = (m * NR + SPAN - 1) / SPAN; r < ((m + 1) * NR + SPAN - 1) / SPAN; ++r)
        if (r < NR) read(cur, 1, r, 1);
      if (m == BAR) {                                               // K-step kt+1 has landed, and nobody reads this one's stage any more
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (DMA) asm volatile("s_waitcnt vmcnt(%0)" : : "n"((NS - 2) * L) : "memory");
        else wait_loads(KT - 2 - kt);
        PIN();
        asm volatile("s_barrier" ::: "memory");
        PIN();
      }
      PIN();
    }
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      mfma(m, 1);
      PIN();
#pragma unroll
      for (int r = (m * NR + SPAN - 1) / SPAN; r < ((m + 1) * NR + SPAN - 1) / SPAN; ++r)
        if (r < NR) read(nxt, 0, r, 0);
      if (DMA) {
#pragma unroll
        for (int n = 0; n < L; ++n)
          if (m == n * NM / L) dma(n, fill);
      }
      PIN();
    }
    if (DMA) b_src += b_step;
  };
#pragma unroll
  for (int t = 0; t < NS; ++t) {
    if (t < KT) {
#pragma unroll
      for (int n = 0; n < L; ++n) dma(n, t * STAGE);
      b_src += b_step;
    }
  }
  PIN();
  wait_loads(KT - 1);                                               // K-step 0 has landed
  PIN();
  asm volatile("s_barrier" ::: "memory");
  PIN();
#pragma unroll
  for (int r = 0; r < NR; ++r) read(smem, 0, r, 0);
  PIN();
  int kt = 0;
#pragma unroll 1
  for (; kt < KT - NS; ++kt) kstep(std::true_type{}, kt);
#pragma unroll 1
  for (; kt < KT; ++kt) kstep(std::false_type{}, kt);               // the last one reads ahead a stage that holds nothing new, for no use
}

// ACT, MODE, GRAD, DUAL: see grouped_gemm_mfma_kernel.
template <int TM, int TN, int NS, int ACT, int MODE, bool GRAD, bool DUAL>
__device__ __forceinline__ void run_piece(char* smem, const Piece& p, uint16_t* out, const uint16_t* pre, uint16_t* pre_out) {
  constexpr int WTM = TM / 2, WTN = TN / 2, RA = WTM / 16, RB = WTN / 16, CPR = WTN / 8, RPS = 64 / CPR;   // rows to a store
  static_assert(TM % 128 == 0 && TN == 128 && NS * (TM + TN) * 128 <= kRingBytes, "loads and swizzles, a unit's LDS");
  const int lane = threadIdx.x & 63, kq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  f32x4 acc[RA][RB];
  if (p.rows > WTM) piece_main_loop<TM, TN, NS, MODE, TM / 32, RA>(smem, p, lane, wave, acc);
  else if (wm == 0) piece_main_loop<TM, TN, NS, MODE, TM / 64, RA>(smem, p, lane, wave, acc);
  else piece_main_loop<TM, TN, NS, MODE, TM / 64, 0>(smem, p, lane, wave, acc);
  const int live = p.rows - wm * WTM;
  if (live <= 0) return;                                            // no barrier follows
  // epilogue as the large tile's: wave w's own [WTM rows][CPR pieces of 8 columns], piece c of row r at c ^ (r % CPR)
  char* wtile = smem + wave * (WTM * WTN * 2);
  const int64_t out_at = p.out + (int64_t)wm * WTM * p.N + wn * WTN;
  auto write_tile = [&](auto raw_tag, uint16_t* dst) {
    constexpr bool RAW = decltype(raw_tag)::value;
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      const int r = i * 16 + (lane & 15);
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = epilogue_act<(GRAD || RAW) ? -1 : ACT>(acc[i][j][u]);
        u32x2 pk;
        pk.x = pack_bf16x2(v[0], v[1]);
        pk.y = pack_bf16x2(v[2], v[3]);
        *LDS_PTR(u32x2, wtile + r * (WTN * 2) + (((2 * j + (kq >> 1)) ^ (r % CPR)) << 4) + 8 * (kq & 1)) = pk;
      }
    }
    constexpr int BATCH = WTM / RPS < 8 ? WTM / RPS : 8;
    for (int it0 = 0; it0 < WTM / RPS; it0 += BATCH) {
      if (it0 * RPS >= live) break;
      uint4 pv[BATCH];
      if (GRAD && !RAW) {                                           // this batch's pre-activations, all loads in flight at once
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
          const int r = (it0 + u) * RPS + lane / CPR, rr = r < live ? r : 0;
          pv[u] = *reinterpret_cast<const uint4*>(pre + out_at + (int64_t)rr * p.N + (((lane % CPR) ^ (rr % CPR)) << 3));
        }
      }
#pragma unroll
      for (int u = 0; u < BATCH; ++u) {
        const int r = (it0 + u) * RPS + lane / CPR;
        u32x4 q = *LDS_PTR(u32x4, wtile + r * (WTN * 2) + ((lane % CPR) << 4));
        if (r >= live) continue;
        if (GRAD && !RAW) {
          float g[8], f[8];
          Vec16<uint16_t>::unpack(__builtin_bit_cast(uint4, q), g);
          Vec16<uint16_t>::unpack(pv[u], f);
#pragma unroll
          for (int v = 0; v < 8; ++v) g[v] = ACT < 0 ? g[v] + f[v] : g[v] * epilogue_act_grad<ACT>(f[v]);
          q = __builtin_bit_cast(u32x4, Vec16<uint16_t>::pack(g));
        }
        *reinterpret_cast<u32x4*>(dst + out_at + (int64_t)r * p.N + (((lane % CPR) ^ (r % CPR)) << 3)) = q;
      }
    }
  };
  if (DUAL) write_tile(std::true_type{}, pre_out);
  write_tile(std::false_type{}, out);
}

}  // namespace
