// The grouped GEMM of ffn_mfma.hip for bf16 products that its large tile does not cover or does not suit and that have the rows and
// columns for tiles of TM x TN: any K and N that are multiples of 8, the layouts kNN, kNT and kTN.  Included by ffn_mfma.hip.
//
//   out[e] = epilogue(A[e] * B[e] + bias[e])
//
// The loop is the large tile's: four waves of TM/2 x TN/2 as tiles of v_mfma_f32_16x16x32_bf16, K in steps of 64 through LDS rings of
// two stages for A and three for B filled by direct global->LDS loads two K-steps ahead, one barrier per K-step, every
// matrix instruction followed by the LDS reads and direct loads that are due there.  What differs is the edges.  Every lane has an
// address of its own for each of its loads: rows past the fill repeat the last live row, columns past N the tile's first piece
// (neither is stored), and in the last K-step the pieces past the end of the reduction come from a piece of zeros: no side buffer,
// no launch to fill it.
//
// 128 x 128: the rings take half of a unit's LDS, so two blocks share it and one's products cover the other's barrier, tile search and epilogue.
// It binds by LDS (a K-step's reads and fills take 660 cycles at the rates measured for them, its products 512) and by the loads' way
// from L2.  Against 128 x 128 as 32 x 32 x 16 instructions on two stages of both operands, product by product (62 to 68 shapes each off and on
// the large tile's grid, 3e8 to 1.5e11 flop): forward 0.94 of the time, with kept pre-activations 0.95, B transposed 0.92, with the act'
// epilogue 0.87 and 0.82, weight gradients of slabs 0.99, gathered 0.92 (slowest 1.10: 125 experts x 76 rows, 512 x 768).  Whole training
// steps: 87913 tokens, 4 experts, 512 x 512 2735 -> 2408 us, 17 x 353 rows, 776 x 1544 309 -> 304 on one board.
//
// LDS layouts: a k-contiguous operand as in the large tile.  A k-slow operand of width W is [64 k][W / 8 pieces]; a transposing
// read takes 32 bytes of each of 4 k rows, and two of its 16-lane blocks, 8 k apart, share a cycle.  Their eight pieces of 32
// bytes cover all 64 banks once if the 4 rows lie in different 64-byte windows modulo 256 (pieces swizzled by 4 (k % 4)) and
// the blocks in different halves of them (2 (k / 8 % 2)).

namespace {

constexpr int ring_bytes(int tm, int tn) { return (2 * tm + 3 * tn) * 128; }
constexpr int divisor_up_to_8(int n) {
  int d = 1;
  for (int i = 2; i <= 8; ++i) d = n % i == 0 ? i : d;
  return d;
}

// GK (kTN): A's k rows (slots) are gathered.
template <int MODE, int TM, int TN, bool GK = false>
__global__ __launch_bounds__(256, 2 * ring_bytes(TM, TN) <= 163840 ? 2 : 1) void grouped_gemm_ring_kernel(const TileArgs p) {
  constexpr bool TRA = MODE == kTN, TRB = MODE != kNT;              // k-slow operands
  constexpr int WTM = TM / 2, WTN = TN / 2, RA = WTM / 16, RB = WTN / 16;
  constexpr int LA = TM / 32, LB = TN / 32;                         // direct loads per wave and K-step
  constexpr int A_STAGE = TM * 128, B_STAGE = TN * 128, B_RING = 2 * A_STAGE;
  constexpr int RING = ring_bytes(TM, TN);
  static_assert(RING <= 163840 && TM * TN * 2 <= RING && TM % 128 == 0 && TN % 128 == 0, "rings fit a unit, the epilogue's transpose the rings, the swizzles the widths");
  __shared__ __attribute__((aligned(1024))) char smem[RING];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave >> 1, wn = wave & 1, kq = lane >> 4;
  int e, mt, nt, rows;
  if (!p.plain) {
    if (!find_tile<TM, MODE == kTN>(blockIdx.x, lane, p.E, p.C, p.counts, p.NT, e, mt, nt, rows)) return;
  } else {
    e = blockIdx.y;
    mt = blockIdx.x / p.NT;
    nt = blockIdx.x % p.NT;
    rows = live_rows_of(e, p.C, p.counts);
  }
  const int64_t m0 = (int64_t)mt * TM, n0 = (int64_t)nt * TN;
  if (m0 >= rows) return;
  int64_t kend = p.K;                                               // k that exist
  if (MODE == kTN && p.kfill) { const int64_t c = p.kfill[e]; kend = c < p.K ? (c > 0 ? c : 0) : p.K; }
  const int KT = kend > 0 ? (int)((kend + 63) / 64) : 1;

  // ---- this lane's direct loads.  k-contiguous: block q * 4 + wave = 8 rows, lane l row + l / 8, position l % 8.  k-slow: pieces in order.
  auto swz_slow = [](int kr) -> int { return (4 * (kr & 3)) ^ (2 * ((kr >> 3) & 1)); };
  auto slow_k = [&](int q, int width) -> int { return ((q * 4 + wave) * 64 + lane) / (width / 8); };
  const int fast_k = ((lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7)) * 8;
  auto slow_source = [&](const uint16_t* base, int64_t ld, int64_t c0, int width, int q) -> const char* {
    const int ppr = width / 8, at = (q * 4 + wave) * 64 + lane, kr = at / ppr;
    const int64_t col = c0 + ((at % ppr) ^ swz_slow(kr)) * 8;
    return (const char*)(base + (int64_t)kr * ld + (col < ld ? col : c0));
  };
  const char* a_ptr[LA];
  const char* b_ptr[LB];
#pragma unroll
  for (int q = 0; q < LA; ++q) {
    if (TRA) {
      a_ptr[q] = slow_source((const uint16_t*)p.A + (GK ? 0 : (int64_t)e * p.K * p.C), p.C, m0, TM, q);
      if (GK) a_ptr[q] -= (int64_t)slow_k(q, TM) * p.C * 2;         // of row 0 of the gathered matrix
    } else {
      int64_t row = m0 + (q * 4 + wave) * 8 + (lane >> 3);
      row = row < rows ? row : rows - 1;                            // rows past the fill repeat the last one
      const uint16_t* base = (const uint16_t*)p.A;
      if (p.gather) {
        const int64_t t = p.gather[(int64_t)e * p.C + row];
        row = t >= 0 && t < p.gather_rows ? t : 0;
      } else {
        base += (int64_t)e * p.C * p.K;
      }
      a_ptr[q] = (const char*)(base + row * p.K + fast_k);
    }
  }
#pragma unroll
  for (int q = 0; q < LB; ++q) {
    const uint16_t* base = (const uint16_t*)p.B + (int64_t)e * p.K * p.N;
    if (TRB) {
      b_ptr[q] = slow_source(base, p.N, n0, TN, q);
    } else {
      const int64_t row = n0 + (q * 4 + wave) * 8 + (lane >> 3);
      b_ptr[q] = (const char*)(base + (row < p.N ? row : p.N - 1) * p.K + fast_k);
    }
  }
  const int64_t a_step = TRA ? 128 * p.C : 128, b_step = TRB ? 128 * (int64_t)p.N : 128;
  const uint32_t smem_addr = (uint32_t)(uintptr_t)LDS_PTR(char, smem);
  const char* zero = (const char*)g_zero_piece;
  // ahead of the loads of the last K-step: what lies past the end of the reduction is read as zeros
  auto end_a = [&](int left) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < LA; ++q) a_ptr[q] = (TRA ? slow_k(q, TM) : fast_k) < left ? a_ptr[q] : zero;
  };
  auto end_b = [&](int left) __attribute__((always_inline)) {
#pragma unroll
    for (int q = 0; q < LB; ++q) b_ptr[q] = (TRB ? slow_k(q, TN) : fast_k) < left ? b_ptr[q] : zero;
  };
  // gathered A: the rows of a K-step are fetched (plain loads) a K-step before its loads go out
  auto gather_fetch = [&](int t, int (&g)[GK ? LA : 1]) __attribute__((always_inline)) {
    if constexpr (GK) {
#pragma unroll
      for (int q = 0; q < LA; ++q) {
        const int64_t slot = (int64_t)t * 64 + slow_k(q, TM);
        g[q] = p.gather[(int64_t)e * p.K + (slot < p.K ? slot : p.K - 1)];
      }
    }
  };
  // and turned into addresses all at once, behind a wait for everything in flight
  const char* a_row[GK ? LA : 1];
  auto gather_resolve = [&](int t, const int (&g)[GK ? LA : 1]) __attribute__((always_inline)) {
    if constexpr (GK) {
#pragma unroll
      for (int q = 0; q < LA; ++q) {
        const char* at = a_ptr[q] + (int64_t)((uint32_t)g[q] < (uint64_t)p.gather_rows ? g[q] : 0) * p.C * 2;
        a_row[q] = (int64_t)t * 64 + slow_k(q, TM) < kend ? at : zero;
      }
    }
  };
  auto dma_a = [&](int q, int t) __attribute__((always_inline)) {
    const uint32_t dst = smem_addr + (t & 1) * A_STAGE + (q * 4 + wave) * 1024;
    if constexpr (GK) {
      global_to_lds_16(a_row[q], dst);
    } else {
      global_to_lds_16(a_ptr[q], dst);
      a_ptr[q] += a_step;
    }
  };
  auto dma_b = [&](int q, int stage) __attribute__((always_inline)) {
    global_to_lds_16(b_ptr[q], smem_addr + B_RING + stage + (q * 4 + wave) * 1024);
    b_ptr[q] += b_step;
  };

  // ---- LDS read offsets of this lane's fragments -----------------------------------------------------------------
  auto read_fast = [&](const char* stage, int w, int t, int s) __attribute__((always_inline)) -> bf16x8 {
    return *LDS_PTR(bf16x8, stage + (w + t * 16 + (lane & 15)) * 128 + (((4 * s + kq) ^ ((lane & 15) >> 1)) << 4));
  };
  auto read_slow = [&](const char* stage, int w, int t, int width, int s, int half) __attribute__((always_inline)) -> short4v {
    const int kr = kq * 8 + ((lane & 15) >> 2), c = w / 8 + 2 * t + ((lane & 3) >> 1);
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        LDS_PTR(short4v, stage + kr * width * 2 + ((c ^ swz_slow(kr)) << 4) + ((lane & 1) << 3) + (32 * s + 4 * half) * width * 2));
  };
  auto join = [](short4v lo, short4v hi) -> bf16x8 {
    return __builtin_bit_cast(bf16x8, (short8v)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  f32x4 acc[RA][RB];
  const int64_t nw = n0 + wn * WTN;                                 // first column of this wave
  const int64_t live = nw < p.N ? rows - m0 - wm * WTM : 0;         // its rows that exist

  auto main_loop = [&](auto ni_tag) __attribute__((always_inline)) {
    constexpr int NI = decltype(ni_tag)::value;                     // 16-row tiles of this wave that are computed
    constexpr int NM = RA * RB;                                     // products per sub-step (two to a K-step)
    constexpr int NRA = TRA ? 2 * RA : RA, NRB = TRB ? 2 * RB : RB, NR = NRA + NRB, PA = TRA ? 2 : 1;
    // The reads of the next sub-step go out behind the first three quarters of a sub-step's products, the barrier is behind seven eighths of sub-step
    // 0, B's loads of the K-step after next before it and A's after it, evenly; with gathered rows both after it.
    constexpr int SPAN = NM * 3 / 4, BAR = NM * 7 / 8;
    bf16x8 fa[2][RA], fb[2][RB];
    // read number r of sub-step s into fragment buffer d: the first of A, B's, then the rest of A's
    auto read = [&](const char* a_stage, const char* b_stage, int s, int r, int d, short4v& lo) __attribute__((always_inline)) {
      if (NI == 0) return;
      if (r >= PA && r < PA + NRB) {
        const int rb = r - PA;
        if (!TRB) fb[d][rb] = read_fast(b_stage, wn * WTN, rb, s);
        else if ((rb & 1) == 0) lo = read_slow(b_stage, wn * WTN, rb >> 1, TN, s, 0);
        else fb[d][rb >> 1] = join(lo, read_slow(b_stage, wn * WTN, rb >> 1, TN, s, 1));
      } else {
        const int ra = r < PA ? r : r - NRB;
        if (!TRA) { if (ra < NI) fa[d][ra] = read_fast(a_stage, wm * WTM, ra, s); }
        else if ((ra & 1) == 0) lo = read_slow(a_stage, wm * WTM, ra >> 1, TM, s, 0);
        else fa[d][ra >> 1] = join(lo, read_slow(a_stage, wm * WTM, ra >> 1, TM, s, 1));
      }
    };
    auto mfma = [&](int m, int d) __attribute__((always_inline)) {
      const int i = m / RB, j = m % RB;
      if (i < NI) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[d][j], fa[d][i], acc[i][j], 0, 0, 0);
    };
    int grow[GK ? LA : 1], grow1[GK ? LA : 1];
    int b_stage = 0;                                                // byte offset of K-step kt's stage in B's ring
    auto kstep = [&](auto dma_tag, int kt) __attribute__((always_inline)) {
      constexpr bool DMA = decltype(dma_tag)::value;                // K-step kt + 2 exists
      const char* a_cur = smem + (kt & 1) * A_STAGE;
      const char* a_nxt = smem + (~kt & 1) * A_STAGE;
      const int b_fill = b_stage == 0 ? 2 * B_STAGE : b_stage - B_STAGE;
      const char* b_cur = smem + B_RING + b_stage;
      b_stage = b_stage == 2 * B_STAGE ? 0 : b_stage + B_STAGE;
      const char* b_nxt = smem + B_RING + b_stage;
      if (DMA) {
        if (kt + 2 == KT - 1) {
          const int left = (int)(kend - (int64_t)(kt + 2) * 64);
          if (!GK) end_a(left);
          end_b(left);
        }
        if (GK) gather_fetch(kt + 2, grow);
        PIN();
      }
      short4v lo;
      auto reads = [&](int m, const char* a, const char* b, int s, int d) __attribute__((always_inline)) {
#pragma unroll
        for (int r = (m * NR + SPAN - 1) / SPAN; r < ((m + 1) * NR + SPAN - 1) / SPAN; ++r)
          if (r < NR) read(a, b, s, r, d, lo);
      };
      auto loads = [&](int m) __attribute__((always_inline)) {
        if (!DMA) return;
        if (GK) {
#pragma unroll
          for (int n = 0; n < LA + LB; ++n)
            if (m == BAR + n * (2 * NM - BAR) / (LA + LB)) { if (n < LA) dma_a(n, kt + 2); else dma_b(n - LA, b_fill); }
          return;
        }
#pragma unroll
        for (int n = 0; n < LB; ++n)
          if (m == n * BAR / LB) dma_b(n, b_fill);
#pragma unroll
        for (int n = 0; n < LA; ++n)
          if (m == BAR + n * (2 * NM - BAR) / LA) dma_a(n, kt + 2);
      };
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        mfma(m, 0);
        PIN();
        reads(m, a_cur, b_cur, 1, 1);
        if (m == BAR) {                                             // K-step kt+1 has landed, though not B's loads of kt+2 behind it
          if (DMA && !GK) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(LB) : "memory");
          else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
          PIN();
          asm volatile("s_barrier" ::: "memory");
          PIN();
          if (GK && DMA) { gather_resolve(kt + 2, grow); PIN(); }
        }
        loads(m);
        PIN();
      }
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        mfma(m, 1);
        PIN();
        reads(m, a_nxt, b_nxt, 0, 0);
        loads(m + NM);
        PIN();
      }
    };
    gather_fetch(0, grow);
    gather_fetch(1, grow1);
    gather_resolve(0, grow);
    if (KT == 1) { if (!GK) end_a((int)kend); end_b((int)kend); }
#pragma unroll
    for (int q = 0; q < LA; ++q) dma_a(q, 0);
#pragma unroll
    for (int q = 0; q < LB; ++q) dma_b(q, 0);
    if (KT > 1) {
      if (KT == 2) { if (!GK) end_a((int)(kend - 64)); end_b((int)(kend - 64)); }
      gather_resolve(1, grow1);
#pragma unroll
      for (int q = 0; q < LA; ++q) dma_a(q, 1);
#pragma unroll
      for (int q = 0; q < LB; ++q) dma_b(q, B_STAGE);
    }
    // accumulators: the bias (register u of tile (i, j) is column 16 j + 4 kq + u of the wave's), or zero
    const uint16_t* bias = MODE == kNN ? (const uint16_t*)p.bias : nullptr;
#pragma unroll
    for (int j = 0; j < RB; ++j) {
      f32x4 b = {0.f, 0.f, 0.f, 0.f};
      if (bias) {
        const int64_t col = nw + j * 16 + 4 * kq;
        const u32x2 v = *reinterpret_cast<const u32x2*>(bias + (int64_t)e * p.N + (col < p.N ? col : n0));
        b = f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xffff0000u), __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xffff0000u)};
      }
#pragma unroll
      for (int i = 0; i < NI; ++i) acc[i][j] = b;
    }
    PIN();
    if (KT > 1) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(LA + LB) : "memory");   // loads return in order: K-step 0 has landed
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    PIN();
    asm volatile("s_barrier" ::: "memory");
    PIN();
    {
      short4v lo;
#pragma unroll
      for (int r = 0; r < NR; ++r) read(smem, smem + B_RING, 0, r, 0, lo);
    }
    PIN();
    int kt = 0;
    for (; kt < KT - 2; ++kt) kstep(std::true_type{}, kt);
#pragma unroll 1
    for (; kt < KT; ++kt) kstep(std::false_type{}, kt);             // the last one reads ahead a stage that holds nothing new, for no use
  };
  const int ni = live <= 0 ? 0 : (live >= WTM ? RA : (int)((live + 15) >> 4));
  constexpr int HALF = (RA + 1) / 2;
  if (MODE != kTN && ni == 0) main_loop(std::integral_constant<int, 0>{});
  else if (MODE != kTN && ni <= HALF) main_loop(std::integral_constant<int, HALF>{});
  else main_loop(std::integral_constant<int, RA>{});
  if (live <= 0) return;                                            // no barrier follows

  // ---- epilogue: through the wave's own piece of LDS, so that stores are 16 bytes per lane and whole row pieces.  Piece c of row r is
  // at c ^ out_swz(r): both accesses spread over all banks.  No direct load is in flight and no wave reads the stages any more, but for what the
  // last K-step reads ahead and nobody uses.
  constexpr int CPR = WTN / 8, STORES = WTM * CPR / 64, BATCH = divisor_up_to_8(STORES);
  static_assert(WTM * CPR % 64 == 0, "whole stores");
  auto out_swz = [](int r) -> int { return r % CPR; };
  char* wtile = smem + wave * (WTM * WTN * 2);
  const int64_t out_at = ((int64_t)e * p.C + m0 + wm * WTM) * p.N + nw;
  auto write_tile = [&](auto act_tag, uint16_t* dst, const uint16_t* pre) __attribute__((always_inline)) {
    constexpr int ACT = decltype(act_tag)::value;
#pragma unroll
    for (int i = 0; i < RA; ++i) {
      if (i >= ni) break;
      const int r = i * 16 + (lane & 15);
#pragma unroll
      for (int j = 0; j < RB; ++j) {
        float v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) v[u] = MODE == kNN ? tile_act<ACT>(acc[i][j][u]) : acc[i][j][u];
        u32x2 pk;
        pk.x = pack_bf16x2(v[0], v[1]);
        pk.y = pack_bf16x2(v[2], v[3]);
        *LDS_PTR(u32x2, wtile + r * (CPR * 16) + (((2 * j + (kq >> 1)) ^ out_swz(r)) << 4) + 8 * (kq & 1)) = pk;
      }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll 1
    for (int it0 = 0; it0 < STORES; it0 += BATCH) {
      if (it0 * 64 / CPR >= live) break;
      uint4 pv[BATCH];
      int64_t at[BATCH];
      bool on[BATCH];
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        const int n = (it0 + b) * 64 + lane, r = n / CPR, c = (n % CPR) ^ out_swz(r);
        on[b] = r < live && nw + c * 8 < p.N;
        at[b] = on[b] ? out_at + (int64_t)r * p.N + c * 8 : out_at;
        if (MODE == kNT && pre) pv[b] = *reinterpret_cast<const uint4*>(pre + at[b]);
      }
#pragma unroll
      for (int b = 0; b < BATCH; ++b) {
        u32x4 q = *LDS_PTR(u32x4, wtile + ((it0 + b) * 64 + lane) * 16);
        if (MODE == kNT && pre) {                                   // times act'(pre), both factors as stored; or plus `pre`
          float g[8], f[8];
          Vec16<uint16_t>::unpack(__builtin_bit_cast(uint4, q), g);
          Vec16<uint16_t>::unpack(pv[b], f);
#pragma unroll
          for (int u = 0; u < 8; ++u) g[u] = ACT < 0 ? g[u] + f[u] : g[u] * tile_act_grad<ACT>(f[u]);
          q = __builtin_bit_cast(u32x4, Vec16<uint16_t>::pack(g));
        }
        if (on[b]) *reinterpret_cast<u32x4*>(dst + at[b]) = q;
      }
    }
    __builtin_amdgcn_wave_barrier();
  };
  uint16_t* out = (uint16_t*)p.out;
  const uint16_t* pre = MODE == kNT ? (const uint16_t*)p.pre : nullptr;
  if (MODE == kNN && p.pre_out) write_tile(std::integral_constant<int, -1>{}, (uint16_t*)p.pre_out, nullptr);
  if (MODE == kTN) write_tile(std::integral_constant<int, -1>{}, out, nullptr);
  else switch (p.act) {
    case MOE_ACT_RELU: write_tile(std::integral_constant<int, MOE_ACT_RELU>{}, out, pre); break;
    case MOE_ACT_GELU: write_tile(std::integral_constant<int, MOE_ACT_GELU>{}, out, pre); break;
    case MOE_ACT_SILU: write_tile(std::integral_constant<int, MOE_ACT_SILU>{}, out, pre); break;
    case MOE_ACT_GELU + kFullAct: write_tile(std::integral_constant<int, MOE_ACT_GELU + kFullAct>{}, out, pre); break;
    case MOE_ACT_SILU + kFullAct: write_tile(std::integral_constant<int, MOE_ACT_SILU + kFullAct>{}, out, pre); break;
    default: write_tile(std::integral_constant<int, -1>{}, out, pre); break;
  }
}

}  // namespace

template <int MODE, int TM, int TN>
static hipError_t launch_ring(TileArgs p, int64_t total, hipStream_t s) {
  dim3 grid;
  if (!tile_launch(p, TM, TN, total, grid)) return hipErrorInvalidValue;
  if (MODE == kTN && p.gather) grouped_gemm_ring_kernel<MODE, TM, TN, MODE == kTN><<<grid, dim3(256), 0, s>>>(p);
  else grouped_gemm_ring_kernel<MODE, TM, TN><<<grid, dim3(256), 0, s>>>(p);
  return hipGetLastError();
}
