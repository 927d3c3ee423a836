// The grouped GEMM of ffn_mfma.hip for what its larger tiles do not cover or do not suit: fp32 storage, and bf16 launches with few
// tiles, with any K and N that are multiples of 8.  Included by ffn_mfma.hip (same helpers, same operand layouts).
//
//   out[e] = epilogue(A[e] * B[e] + bias[e]) in the layouts kNN, kNT and kTN, bf16 (v_mfma_f32_32x32x16_bf16) or fp32
//   (v_mfma_f32_32x32x2_f32: full fp32 products and sums), fp32 accumulation.
//
// One K-step is 128 bytes of k (64 bf16, 32 fp32), staged through an NS-deep LDS ring by direct global->LDS loads with an
// address per lane, so that edges cost nothing inside: rows past the fill repeat the last live row, columns past N the
// tile's first piece (neither is stored), and the pieces of the last K-step that lie past the end of the reduction come
// from a 16-byte piece of zeros.  No operand is copied, padded or transposed in memory.  In bytes the LDS layouts and their
// swizzles are the same for both types:
//   k-contiguous operand: [rows][8 pieces of 16 bytes], piece g of row r at position g ^ ((r / 2) % 8)  (ds_read_b128)
//   k-slow operand:       [k rows][width], bf16 pieces swizzled for ds_read_b64_tr_b16, fp32 read as single words
// Several blocks share a compute unit (72 KB of LDS or less each), so that one block's matrix instructions cover another's
// barrier, load latency, tile search and epilogue; what is left binds by LDS reads and, for few tiles, by how evenly they divide
// among the units.
//
// What it replaced was an fp32 FMA kernel on operands transposed and padded in memory, at 12 TFLOP/s in either type.
// Measured, training step of 17 experts x 353 rows, M = 776, H = 1544, bf16: the six products 645-700 us -> 35-57 us each
// (33-43 on the 128 x 128 tile of ffn_ring.h, which takes them now), step 5060 -> 340 us.  8 experts x 1024 rows, M = 512, H = 1024, fp32: products 166-228 us -> 72-95 us
// (117 TFLOP/s in the weight gradients; fp32 matrix peak 157), step 1585 -> 603 us.  8 experts x 4 rows, M = H = 2048, bf16: 29 us
// on the large tile -> 13 us (67 MB of weights: 5.1 TB/s), layer 121 -> 51 us.

namespace {

// Waits until at most min(later, MOST) K-steps' loads, L of them each, are outstanding.
template <int MOST, int L> __device__ __forceinline__ void wait_for_loads(int later) {
  if constexpr (MOST > 0) {
    if (later < MOST) { wait_for_loads<MOST - 1, L>(later); return; }
  }
  asm volatile("s_waitcnt vmcnt(%0)" : : "n"(MOST * L) : "memory");
}

// GK (kTN): A's k rows (slots) are gathered; the row numbers of a K-step are fetched a K-step before its loads go out.
// PART (kTN): one long product cut along its reduction: "expert" e reduces k = e K .. e K + K - 1, and the sums leave as fp32.
// In fp32 a chain of products ends after 64 k and the chains' sums are added up apart, as they were before the slices grew past 64:
// the error of dWg in fp32 gates, 2-norm of the result, tokens of one sign: 1000 tokens 2.6e-7 with chains as long as the slice,
// 1.4e-7 so; 131072 tokens 6.8e-7 and 1.7e-7.  Results rounded to bf16 show no difference (at most 7e-4 of dWg rounds the other
// way either way).
// STREAM: B is loaded as data that is read once.
// KS: waves that share a tile of one wave along its reduction, wave w taking K-steps w, w + KS and so on through stages of its own
// (no barrier until their sums meet, which the first wave adds up in order).  For fp32 launches of few tiles, whose time is one chain
// of matrix instructions per wave on a part of the units: see fp32_split.  Two stages (64 KB, two blocks to a unit): three or four
// leave room for one block, 4 experts x 256 rows, 256 x 512, two products: 15.4 us against 19.4 and 19.7.
template <typename ET, int MODE, int BM, int BN, int WR, int WC, int NS, bool GK = false, bool PART = false, bool STREAM = false, int KS = 1>
__global__ __launch_bounds__(WR * WC * KS * 64, 2) void grouped_gemm_tile_kernel(const TileArgs p) {
  constexpr int ES = (int)sizeof(ET), EC = 16 / ES;                 // elements per 16-byte piece
  constexpr int BKE = 128 / ES;                                     // k per K-step
  constexpr bool BF16 = ES == 2;
  constexpr bool TRA = MODE == kTN, TRB = MODE != kNT;              // k-slow operands
  constexpr int NW = WR * WC;
  constexpr int WTM = BM / WR, WTN = BN / WC, TI = WTM / 32, TJ = WTN / 32;
  constexpr int A_BYTES = BM * 128, STAGE = (BM + BN) * 128;
  constexpr int LA = A_BYTES / (NW * 1024), LB = BN * 128 / (NW * 1024);   // direct loads per wave and K-step
  static_assert(LA >= 1 && LB >= 1 && TI >= 1 && TJ >= 1, "every wave loads and owns something");
  constexpr bool BF16O = BF16 && !PART;                             // type of the results
  constexpr int OS = BF16O ? 2 : 4, OC = 16 / OS;
  static_assert(NW * WTM * WTN * OS <= NS * STAGE, "the epilogue's transpose fits into the stages");
  static_assert(KS == 1 || (NW == 1 && TI == 1 && TJ == 1 && !GK && !PART && KS * WTM * WTN * 4 <= KS * NS * STAGE), "split: one 32 x 32 tile");
  __shared__ __attribute__((aligned(1024))) char smem_all[KS * NS * STAGE];

  const int lane = threadIdx.x & 63;
  const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wave = KS > 1 ? 0 : wave_id, part = KS > 1 ? wave_id : 0;   // wave of the tile; its share of the reduction
  char* const smem = smem_all + part * (NS * STAGE);
  const int wm = wave / WC, wn = wave % WC, kg = lane >> 5;

  // ---- which tile: the search of the large kernel, or plain numbering where that does not do ---------------------
  int e, mt, nt, rows;
  if (!p.plain) {
    if (!find_tile<BM, MODE == kTN>(blockIdx.x, lane, p.E, p.C, p.counts, p.NT, e, mt, nt, rows)) return;
  } else {
    e = blockIdx.y;
    mt = blockIdx.x / p.NT;
    nt = blockIdx.x % p.NT;
    rows = live_rows_of(e, p.C, p.counts);
  }
  const int64_t m0 = (int64_t)mt * BM;
  if (m0 >= rows) return;
  const int64_t n0 = (int64_t)nt * BN;
  int64_t kend = p.K;                                               // k that exist
  if (MODE == kTN && p.kfill) { const int64_t c = p.kfill[e]; kend = c < p.K ? (c > 0 ? c : 0) : p.K; }
  if (PART) { const int64_t left = p.ktotal - (int64_t)e * p.K; kend = left < p.K ? (left > 0 ? left : 0) : p.K; }
  const int KT_all = kend > 0 ? (int)((kend + BKE - 1) / BKE) : 1;
  const int KT = KS > 1 ? (KT_all - part + KS - 1) / KS : KT_all;   // K-steps of this wave (none where there are fewer than waves)

  // ---- this lane's direct loads: address at K-step 0, and k of its piece (to tell what lies past the end) ---------------
  const char* a_ptr[LA];
  const char* b_ptr[LB];
  int a_k[LA], b_k[LB];
  // k-contiguous: block i*NW + wave = 8 rows, lane l row +l/8, position l%8.   k-slow: PB bytes per k row.
  auto swz_slow = [](int kr, int width_bytes) -> int {              // bf16 only: see tr_off
    return width_bytes >= 256 ? 4 * (kr & 3) : (width_bytes == 128 ? 4 * ((kr >> 1) & 1) : 0);
  };
  auto slow_source = [&](const char* base, int64_t ld, int64_t c0, int width, int i, int& k_out) -> const char* {
    const int pb = width * ES, ppr = pb / 16, rpb = 1024 / pb;      // bytes and pieces per k row, k rows per 1 KB block
    const int kr = (i * NW + wave) * rpb + lane / ppr;
    const int c = (lane % ppr) ^ (BF16 ? swz_slow(kr, pb) : 0);
    const int64_t col = c0 + c * EC;
    k_out = kr;
    return base + ((int64_t)kr * ld + (col < ld ? col : c0)) * ES;  // columns past the end: any piece of the row
  };
  auto fast_source = [&](const char* base, int64_t ld, int64_t row, int i, int& k_out) -> const char* {
    const int r = (i * NW + wave) * 8 + (lane >> 3);
    const int g = (lane & 7) ^ ((r >> 1) & 7);
    k_out = g * EC;
    return base + (row * ld + g * EC) * ES;
  };
#pragma unroll
  for (int i = 0; i < LA; ++i) {
    if (TRA) {
      const char* base = (const char*)p.A + (GK ? 0 : (int64_t)e * p.K * p.C * ES);
      a_ptr[i] = slow_source(base, p.C, m0, BM, i, a_k[i]);
      if (GK) a_ptr[i] -= (int64_t)a_k[i] * p.C * ES;              // row 0 of the gathered matrix
    } else {
      int64_t row = m0 + (i * NW + wave) * 8 + (lane >> 3);
      row = row < rows ? row : rows - 1;                            // rows past the fill repeat the last one
      if (p.gather) {
        const int64_t t = p.gather[(int64_t)e * p.C + row];
        a_ptr[i] = fast_source((const char*)p.A, p.K, t >= 0 && t < p.gather_rows ? t : 0, i, a_k[i]);
      } else {
        a_ptr[i] = fast_source((const char*)p.A + (int64_t)e * p.C * p.K * ES, p.K, row, i, a_k[i]);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < LB; ++i) {
    const char* base = (const char*)p.B + (int64_t)e * p.K * p.N * ES;
    if (TRB) {
      b_ptr[i] = slow_source(base, p.N, n0, BN, i, b_k[i]);
    } else {
      const int64_t row = n0 + (i * NW + wave) * 8 + (lane >> 3);
      b_ptr[i] = fast_source(base, p.K, row < p.N ? row : p.N - 1, i, b_k[i]);
    }
  }
  const int64_t a_one = TRA ? (int64_t)BKE * p.C * ES : 128, b_one = TRB ? (int64_t)BKE * p.N * ES : 128;
  const int64_t a_step = a_one * KS, b_step = b_one * KS;
  if (KS > 1) {
#pragma unroll
    for (int i = 0; i < LA; ++i) a_ptr[i] += a_one * part;
#pragma unroll
    for (int i = 0; i < LB; ++i) b_ptr[i] += b_one * part;
  }
  const uint32_t smem_addr = (uint32_t)(uintptr_t)LDS_PTR(char, smem);
  const char* zero = (const char*)g_zero_piece;
  int grow[GK ? LA : 1];                                            // rows of the next K-step to load
  auto fetch_rows = [&](int t, int (&g)[GK ? LA : 1]) __attribute__((always_inline)) {
    if constexpr (GK) {
#pragma unroll
      for (int i = 0; i < LA; ++i) {
        const int64_t slot = (int64_t)t * BKE + a_k[i];
        g[i] = p.gather[(int64_t)e * p.K + (slot < p.K ? slot : p.K - 1)];
      }
    }
  };
  auto a_source = [&](int i, const int (&g)[GK ? LA : 1]) __attribute__((always_inline)) -> const char* {
    if constexpr (GK) return a_ptr[i] + (int64_t)((uint32_t)g[i] < (uint64_t)p.gather_rows ? g[i] : 0) * p.C * ES;
    else return a_ptr[i];
  };
  auto issue_whole = [&](int t, const int (&g)[GK ? LA : 1]) __attribute__((always_inline)) {   // K-step t -> stage t % NS; t ascends by one per call
    const uint32_t dst = smem_addr + (uint32_t)((t % NS) * STAGE);
#pragma unroll
    for (int i = 0; i < LA; ++i) { global_to_lds_16(a_source(i, g), dst + (i * NW + wave) * 1024); if (!GK) a_ptr[i] += a_step; }
#pragma unroll
    for (int i = 0; i < LB; ++i) { global_to_lds_16<STREAM>(b_ptr[i], dst + A_BYTES + (i * NW + wave) * 1024); b_ptr[i] += b_step; }
  };
  auto issue = [&](int t, const int (&g)[GK ? LA : 1]) __attribute__((always_inline)) {   // the same, with zeros past the end of the reduction
    if (t * KS + part < KT_all - 1) { issue_whole(t, g); return; }
    const uint32_t dst = smem_addr + (uint32_t)((t % NS) * STAGE);
    const int left = (int)(kend - (int64_t)(t * KS + part) * BKE);
#pragma unroll
    for (int i = 0; i < LA; ++i) global_to_lds_16(a_k[i] < left ? a_source(i, g) : zero, dst + (i * NW + wave) * 1024);
#pragma unroll
    for (int i = 0; i < LB; ++i) global_to_lds_16(b_k[i] < left ? b_ptr[i] : zero, dst + A_BYTES + (i * NW + wave) * 1024);
  };

  // ---- LDS read offsets of this lane's fragments (sub-tile 0; the others are constants apart) ---------------------------
  const int swz = ((lane & 31) >> 1) & 7;
  auto read_fast = [&](const char* tile, int w, int t, int s) -> u32x4 {   // pieces 2 s + kg of row w*.. + 32 t + lane % 32
    return *LDS_PTR(u32x4, tile + (w + t * 32 + (lane & 31)) * 128 + (((2 * s + kg) ^ swz) << 4));
  };
  auto read_slow = [&](const char* tile, int w, int t, int width, int s) -> u32x4 {
    if constexpr (BF16) {
      const int pb = width * 2, kr = (lane & 15) >> 2;
      const int c = w / 8 + t * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
      const char* at = tile + (kg * 8 + kr) * pb + ((c ^ swz_slow(kr, pb)) << 4) + ((lane & 1) << 3);
      const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4v, at + 16 * s * pb));
      const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(LDS_PTR(short4v, at + (16 * s + 4) * pb));
      return __builtin_bit_cast(u32x4, (short8v)__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
    } else {
      u32x4 v;
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = *LDS_PTR(uint32_t, tile + (8 * s + 4 * kg + u) * width * 4 + (w + t * 32 + (lane & 31)) * 4);
      return v;
    }
  };

  // ---- accumulators: the bias (register 4 g + u of tile (i, j) is column 32 j + 8 g + 4 kg + u of the wave's), or zero; its
  // loads go out ahead of the first K-steps' and are used behind them
  using Raw4 = std::conditional_t<BF16, u32x2, u32x4>;
  Raw4 braw[TJ][4];
  const bool has_bias = MODE == kNN && p.bias != nullptr && part == 0;
  const int64_t bcol = n0 + wn * WTN + 4 * kg;
  if (has_bias) {
    const ET* be = (const ET*)p.bias + (int64_t)e * p.N;
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int64_t col = bcol + j * 32 + 8 * g;
        braw[j][g] = *reinterpret_cast<const Raw4*>(be + (col < p.N ? col : n0));
      }
  }
  int first_rows[NS][GK ? LA : 1];
#pragma unroll
  for (int t = 0; t < NS; ++t) fetch_rows(t, first_rows[t]);
#pragma unroll
  for (int t = 0; t < NS; ++t)
    if (t < KT) issue(t, first_rows[t]);
  fetch_rows(NS, grow);
  f32x16 acc[TI][TJ];
#pragma unroll
  for (int j = 0; j < TJ; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float b = 0.f;
        if (has_bias) {
          if constexpr (BF16) b = __uint_as_float((u & 1) ? braw[j][g][u >> 1] & 0xffff0000u : braw[j][g][u >> 1] << 16);
          else b = __uint_as_float(braw[j][g][u]);
        }
#pragma unroll
        for (int i = 0; i < TI; ++i) acc[i][j][4 * g + u] = b;
      }

  constexpr bool CHAINS = PART && !BF16;
  f32x16 chains[CHAINS ? TI : 1][CHAINS ? TJ : 1];                  // sums of the chains that have ended
  auto end_chain = [&]() __attribute__((always_inline)) {
    if constexpr (CHAINS) {
#pragma unroll
      for (int i = 0; i < TI; ++i)
#pragma unroll
        for (int j = 0; j < TJ; ++j)
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            chains[i][j][u] += acc[i][j][u];
            acc[i][j][u] = 0.f;
          }
    }
  };
  if constexpr (CHAINS) {
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int u = 0; u < 16; ++u) chains[i][j][u] = 0.f;
  }

  // 32-row sub-tiles of this wave that hold real rows
  const int64_t live = rows - m0 - wm * WTM;
  const int ni = live <= 0 ? 0 : (live >= WTM ? TI : (int)((live + 31) >> 5));

  // Fragments are read one sub-step (a quarter of a K-step) ahead of their MFMAs, across K-steps too: the barrier that hands
  // a stage over sits ahead of the last sub-step's MFMAs, when every read of the stage is done, and the stage is refilled
  // right behind it with the K-step NS ahead.
  auto main_loop = [&](auto ni_tag) __attribute__((always_inline)) {
    constexpr int NI = decltype(ni_tag)::value;
    u32x4 fa[2][TI], fb[2][TJ];                                     // bf16: 8 k; fp32: k = 8 s + 4 kg + u in register u
    auto read = [&](int d, const char* sa, int s) __attribute__((always_inline)) {
      const char* sb = sa + A_BYTES;
#pragma unroll
      for (int i = 0; i < NI; ++i) fa[d][i] = TRA ? read_slow(sa, wm * WTM, i, BM, s) : read_fast(sa, wm * WTM, i, s);
#pragma unroll
      for (int j = 0; j < TJ; ++j)
        if (NI > 0) fb[d][j] = TRB ? read_slow(sb, wn * WTN, j, BN, s) : read_fast(sb, wn * WTN, j, s);
    };
    auto mfmas = [&](int d) __attribute__((always_inline)) {
      if constexpr (BF16) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
          for (int j = 0; j < TJ; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fb[d][j]), __builtin_bit_cast(bf16x8, fa[d][i]), acc[i][j], 0, 0, 0);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int j = 0; j < TJ; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fb[d][j][u]), __uint_as_float(fa[d][i][u]), acc[i][j], 0, 0, 0);
      }
    };
    auto kstep = [&](auto steady_tag, int kt) __attribute__((always_inline)) {
      constexpr bool STEADY = decltype(steady_tag)::value;          // K-step kt + NS exists and is not the last
      const char* cur = smem + (kt % NS) * STAGE;
#pragma unroll
      for (int s = 0; s < 3; ++s) {
        read((s + 1) & 1, cur, s + 1);
        PIN();
        mfmas(s & 1);
        PIN();
      }
      if (STEADY || kt + 1 < KT) {
        if (STEADY) wait_for_loads<NS - 2, LA + LB>(NS);            // K-step kt + 1 has landed, later ones may be under way
        else wait_for_loads<NS - 2, LA + LB>(KT - 2 - kt);
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // this wave's reads of K-step kt are done
        PIN();
        if (KS == 1) asm volatile("s_barrier" ::: "memory");
        PIN();
        if (STEADY) issue_whole(kt + NS, grow);
        else if (kt + NS < KT) issue(kt + NS, grow);
        if (GK) { fetch_rows(kt + NS + 1, grow); PIN(); }
        read(0, smem + ((kt + 1) % NS) * STAGE, 0);
        PIN();
      }
      mfmas(1);
      PIN();
    };
    wait_for_loads<NS - 1, LA + LB>(KT - 1);
    PIN();
    if (KS == 1) asm volatile("s_barrier" ::: "memory");
    PIN();
    read(0, smem, 0);
    PIN();
    int kt = 0;
    for (; kt + NS < KT - 1; ++kt) {
      kstep(std::true_type{}, kt);
      if (CHAINS && kt * BKE % 64 + BKE == 64) end_chain();
    }
    for (; kt < KT; ++kt) {
      kstep(std::false_type{}, kt);
      if (CHAINS && (kt * BKE % 64 + BKE == 64 || kt == KT - 1)) end_chain();
    }
  };
  if (ni == TI) main_loop(std::integral_constant<int, TI>{});
  else if (TI > 1 && ni == 1) main_loop(std::integral_constant<int, 1>{});
  else main_loop(std::integral_constant<int, 0>{});
  static_assert(TI <= 2, "ragged waves are instantiated for 0 and 1 live sub-tiles");

  // ---- epilogue: the wave's tile goes through its own piece of LDS, so that stores are 16 bytes per lane and whole row
  // pieces; piece c of row r sits at position c ^ (r % pieces per row).
  __syncthreads();                                                  // the stages are done with
  if constexpr (KS > 1) {                                           // the parts' sums, 4 KB each, behind the first wave's tile
    char* sums = smem_all + lane * 16;
    if (part > 0) {
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *LDS_PTR(u32x4, sums + part * 4096 + g * 1024) = u32x4{__float_as_uint(acc[0][0][4 * g]), __float_as_uint(acc[0][0][4 * g + 1]),
                                                               __float_as_uint(acc[0][0][4 * g + 2]), __float_as_uint(acc[0][0][4 * g + 3])};
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int w = 1; w < KS; ++w)
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const u32x4 q = *LDS_PTR(u32x4, sums + w * 4096 + g * 1024);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[0][0][4 * g + u] += __uint_as_float(q[u]);
      }
  }
  constexpr int CPR = WTN * OS / 16, RPI = 64 / CPR;                // pieces per row, rows per store
  char* wtile = smem + wave * (WTM * WTN * OS);
  const int64_t nw = n0 + wn * WTN;
  const int64_t out_at = ((int64_t)e * p.C + m0 + wm * WTM) * p.N + nw;
  using OT = std::conditional_t<BF16O, uint16_t, float>;
  auto write_tile = [&](auto act_tag, OT* dst, const OT* pre) __attribute__((always_inline)) {
    constexpr int ACT = decltype(act_tag)::value;
#pragma unroll
    for (int i = 0; i < TI; ++i) {
      const int r = i * 32 + (lane & 31);
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          float v[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            v[u] = CHAINS ? chains[CHAINS ? i : 0][CHAINS ? j : 0][4 * g + u] : acc[i][j][4 * g + u];
            if (ACT >= 0 && !pre) v[u] = BF16O ? tile_act<ACT>(v[u]) : apply_act(v[u], ACT);
          }
          if constexpr (BF16O) {
            u32x2 pk;
            pk.x = pack_bf16x2(v[0], v[1]);
            pk.y = pack_bf16x2(v[2], v[3]);
            *LDS_PTR(u32x2, wtile + r * (CPR * 16) + (((4 * j + g) ^ (r % CPR)) << 4) + 8 * kg) = pk;
          } else {
            const u32x4 pk = {__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])};
            *LDS_PTR(u32x4, wtile + r * (CPR * 16) + (((8 * j + 2 * g + kg) ^ (r % CPR)) << 4)) = pk;
          }
        }
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int it = 0; it < WTM / RPI; ++it) {
      const int r = it * RPI + lane / CPR;
      const int ch = (lane % CPR) ^ (r % CPR);
      u32x4 q = *LDS_PTR(u32x4, wtile + r * (CPR * 16) + ((lane % CPR) << 4));
      if (r < live && nw + ch * OC < p.N) {
        const int64_t at = out_at + (int64_t)r * p.N + ch * OC;
        if (pre) {                                                  // times act'(pre), both factors as stored; or plus `pre`
          float g[OC], pv[OC];
          Vec16<OT>::unpack(__builtin_bit_cast(uint4, q), g);
          Vec16<OT>::unpack(*reinterpret_cast<const uint4*>(pre + at), pv);
#pragma unroll
          for (int u = 0; u < OC; ++u) g[u] = ACT < 0 ? g[u] + pv[u] : g[u] * (BF16O ? tile_act_grad<ACT>(pv[u]) : apply_act_grad(pv[u], ACT));
          q = __builtin_bit_cast(u32x4, Vec16<OT>::pack(g));
        }
        *reinterpret_cast<u32x4*>(dst + at) = q;
      }
    }
    __builtin_amdgcn_wave_barrier();
  };
  OT* out = (OT*)p.out;
  const OT* pre = MODE == kNT ? (const OT*)p.pre : nullptr;
  if (MODE == kNN && p.pre_out) write_tile(std::integral_constant<int, -1>{}, (OT*)p.pre_out, nullptr);
  if (MODE == kTN) write_tile(std::integral_constant<int, -1>{}, out, nullptr);
  else switch (p.act) {
    case MOE_ACT_RELU: write_tile(std::integral_constant<int, MOE_ACT_RELU>{}, out, pre); break;
    case MOE_ACT_GELU: write_tile(std::integral_constant<int, MOE_ACT_GELU>{}, out, pre); break;
    case MOE_ACT_SILU: write_tile(std::integral_constant<int, MOE_ACT_SILU>{}, out, pre); break;
    case MOE_ACT_GELU + kFullAct: if (BF16O) write_tile(std::integral_constant<int, MOE_ACT_GELU + kFullAct>{}, out, pre); break;
    case MOE_ACT_SILU + kFullAct: if (BF16O) write_tile(std::integral_constant<int, MOE_ACT_SILU + kFullAct>{}, out, pre); break;
    default: write_tile(std::integral_constant<int, -1>{}, out, pre); break;
  }
}

}  // namespace

template <typename ET, int MODE, int BM, int BN, int NS, bool STREAM = false, int KS = 1>
static hipError_t launch_tile(TileArgs p, int64_t total, hipStream_t s) {
  dim3 grid;
  if (!tile_launch(p, BM, BN, total, grid)) return hipErrorInvalidValue;
  if constexpr (MODE == kTN) {
    if (p.gather) {
      grouped_gemm_tile_kernel<ET, MODE, BM, BN, 2, 2, NS, true><<<grid, dim3(256), 0, s>>>(p);
      return hipGetLastError();
    }
  }
  constexpr int W = KS > 1 ? 1 : 2;
  grouped_gemm_tile_kernel<ET, MODE, BM, BN, W, W, NS, false, false, STREAM, KS><<<grid, dim3(256), 0, s>>>(p);
  return hipGetLastError();
}

// The launches below the large tile (`total`: rows of all experts that exist, at most).  fp32: the matrix instruction is 16 times slower, loads hardly matter, and the finest
// tile divides best (64 x 64, five blocks per unit: within 2-4 % of the best of four shapes over 442 launches), but for launches too
// small to fill the chip with it (fp32_split).
template <int MODE>
static hipError_t launch_small(int dtype, Tile tile, const TileArgs& p, int64_t total, hipStream_t s) {
  if constexpr (MODE != kTN) {
    if (dtype == MOE_F32 && fp32_split(p.E, p.C, p.K, p.N)) return launch_tile<float, MODE, kSplitTile, kSplitTile, 2, false, kSplitParts>(p, total, s);
  }
  if (dtype == MOE_F32) return launch_tile<float, MODE, 64, 64, 2>(p, total, s);
  if constexpr (MODE != kTN) {
    switch (tile) {
      case Tile::k64: return launch_tile<uint16_t, MODE, 64, 64, 3>(p, total, s);
      case Tile::k64x128: return launch_tile<uint16_t, MODE, 64, 128, 3>(p, total, s);
      case Tile::k64_stream: return launch_tile<uint16_t, MODE, 64, 64, 4, true>(p, total, s);
      case Tile::k64x128_stream: return launch_tile<uint16_t, MODE, 64, 128, 3, true>(p, total, s);
      default: break;
    }
  }
  return launch_ring<MODE, 128, 128>(p, total, s);
}
