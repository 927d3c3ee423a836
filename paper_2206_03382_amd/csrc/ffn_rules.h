// Which kernel and which grid a product of the grouped GEMM (ffn_mfma.hip) takes: plain host arithmetic on sizes, kept apart
// from the kernels so that a test can ask it without a GPU.
#pragma once
#include <math.h>
#include <stdint.h>

#ifdef __HIPCC__
#define MOE_HOST_DEVICE __host__ __device__
#else
#define MOE_HOST_DEVICE
#endif

namespace moe {

constexpr int kNN = 0, kNT = 1, kTN = 2;    // operand layouts, see the head of ffn_mfma.hip
constexpr int kLargeTile = 256, kLargeK = 64;   // rows and columns of the large tile, its K-step
constexpr int kMaxExperts = 512;            // the tile search keeps one register per 64 experts
constexpr int64_t kMaxBlocks = (int64_t)1 << 24;   // of 256 threads, in a grid dimension: launches beyond 2^32 threads run cut short

static inline int64_t tiles_in(int64_t n, int64_t tile) { return (n + tile - 1) / tile; }

// A weight-gradient product (kTN) reduces over an expert's slots: K-steps of 64 slots, the last one (whole or not) read
// from the side buffers, which also covers an expert without any slot (one K-step of zeros).
MOE_HOST_DEVICE inline int slot_ksteps(int64_t fill) { return fill > 0 ? (int)((fill + kLargeK - 1) / kLargeK) : 1; }

struct TileAt { int e, mt, nt; };           // expert, row tile, column tile

// Tile q of the rows x NT ones of expert e: by blocks of 8 tile columns and, inside a block, row by row, so that 32 consecutive ones are 4 row
// tiles x 8 column tiles that share A rows and B columns.
MOE_HOST_DEVICE inline TileAt tile_in_expert(int e, int q, int rows, int NT) {
  const int full = (NT / 8) * rows * 8;                             // its tiles in full 8-column blocks
  if (q < full) return {e, (q % (rows * 8)) / 8, (q / (rows * 8)) * 8 + q % 8};
  const int w = NT % 8, r = q - full;
  return {e, r / w, (NT / 8) * 8 + r % w};
}

// How the other launches (kNN, kNT), whose experts hold different numbers of row tiles, are numbered; the search by a wave is find_tile in
// ffn_device.h.  Hardware deals blocks round-robin: block b runs on XCD b % 8, as the b / 8-th of its tiles, and the tiles that an XCD holds at one
// time should be neighbours in its own L2.  Large launches deal whole groups of an expert's tiles to the XCDs in turn, as many as there are full
// ones for all eight.  Everything left (all of a smaller launch) is one sequence, expert by expert, cut into 8 runs of
// equal length (to a tile), one to an XCD: even whatever the fills are.  Groups of 8 to 32 tiles dealt throughout, short ones last,
// left XCDs with up to a round of tiles more than others: 17 experts x 14 tiles 42 us, 24 so; ViT layer of 32 experts x 784 rows 382 ->
// 355, training step of 17 x 353 rows 314 -> 291.  Runs of an eighth for every launch cost where XCDs next to each other
// share what they read beyond their L2: 8 experts x 4096 rows, 2048 x 2048 (1088 tiles) layer 592 us in groups, 604 in eighths, 603 in
// rounds of 32 cut without regard to experts, 0.996 of the rate in groups so.
//
// A group is what an XCD's 32 units hold at one time: 32 tiles of the large tile and of the smaller ones, 64 of the half tile, of which two blocks
// share a unit (kHalfGroupShift).  Groups of 32 half tiles brought 1.4 times as many panels of A and B into an L2 (32 experts x 784 rows, 3072
// columns; 1.7 times for 2000 rows, 2048 columns).  Layers, 32 and 64 to a group: 43811 tokens, 64 experts, top-4, 512 x 3840 1567 and 1528 us; 29598, 64, top-8,
// 256 x 256 247 and 242; ViT 347.8 and 347.0; with 256 k, where panels are small, also slower: 41617, 32, top-1, 256 x 2560 240 and 243.
// Groups are dealt from four rounds of the chip on, on the large and on the half tile.  (17 experts x 353 rows on 128 x 128, 663 tiles: step 328 us in
// rounds of 32, 309 in eighths.)  Experts of fewer than four row tiles on average stay in eighths.  Over 25 layers and steps of 1 to 6 row tiles
// that is 0.1 % faster on average: 2 % for 64 experts x 256 rows, 1000 x 2056, 48 x 188, 1544 x 2056 and 96 x 417, 768 x 1544, 2 % slower for
// a step of 64 x 125, 1000 x 2000 and for 96 imbalanced ones, 768 x 1544.
constexpr int kGroupShift = 5, kHalfGroupShift = 1, kDealtTiles = 1024;
MOE_HOST_DEVICE inline bool deals_groups(int live, int E, int NT, int shift) { return live >= kDealtTiles << shift && live >= 4 * E * NT; }

// With an imbalanced gate an even share of the tiles is no even share of the work: the experts that fill their capacity have whole row tiles, the
// others one that is nearly empty, and a run may hold only ones or only others.  Where an expert has more than 1.5 times the mean
// rows, the large and the half tile therefore number the row tiles that are filled to more than half first and cut the short ones (an
// expert's last one, at most) into runs of their own, which come after.  Zipf-shaped gates, products without and with: 64 experts x 550 rows, 2560 x
// 1024 94.1 and 80.8 us; 128 experts, 512 x 2048 27.2 and 21.4; 8 x 3000, 2048 x 1536 96.5 and 78.3; training step of the last 562
// and 535; the slowest 8 x 4096, 2048 x 2048 120.6 and 128.1 (step 761 and 786).  An even gate keeps them where they are: next to the
// expert's other tiles they find its weights in the L2 (32 experts x 166 rows, 1856 x 3840 131 us, 183 apart; ViT 328 and 343).  So do the
// smaller tiles, which read more weights for a product (128 x 128, 16 x 750 rows, 1000 x 2000 54.6 and 61.0).
// The exception are few short tiles that alone open another round of the chip, the second or third: 32 experts x 500 rows, 2048 x 2048, layer 392
// and 361 us; 64 x 246, 768 x 1024 145 and 135; 16 x 237, 3072 x 4096 340 and 321; the slowest of 14 such, 64 x 121, 2560 x 3840, 723 and 738.
// Many of them cost what they read (48 x 160, 2304 x 2816, as many shorts as others: 431 and 568), and with more rounds there is no difference.
MOE_HOST_DEVICE inline bool opens_a_round(int tall, int all, int shift) {
  const int places = 256 << shift;
  return (all - tall) * 3 <= tall && tall <= 2 * places && (tall + places - 1) / places < (all + places - 1) / places;
}
MOE_HOST_DEVICE inline bool may_open_a_round(int all, int shift) { return all <= 3 * (256 << shift); }   // spares larger launches the count: 4/3 of two rounds, at most
MOE_HOST_DEVICE inline bool far_above_mean(int rows, int E, int all_rows) { return 2.0f * (float)rows * (float)E > 3.0f * (float)all_rows; }
MOE_HOST_DEVICE inline int tall_row_tiles(int rows, int tile_rows, bool apart) { return (rows + (apart ? tile_rows / 2 : tile_rows) - 1) / tile_rows; }

enum TilePart { kDealtTile, kLeftTile, kShortTile, kNoTile };
struct TileSpot { TilePart part; int at; }; // kDealtTile: number of the group among all; else of the tile among those left, or the short ones
// tall, shorts: tiles of either kind; gs: log2 of a group's tiles, of which each XCD takes `rounds` groups.
MOE_HOST_DEVICE inline TileSpot tile_spot(int b, int tall, int shorts, int rounds, int gs) {
  const int x = b % 8, i = b / 8, dealt = rounds << gs;
  if (i < dealt) return {kDealtTile, (i >> gs) * 8 + x};
  const int left = tall - 8 * dealt, first = x * left / 8, own = (x + 1) * left / 8 - first, j = i - dealt;
  if (j < own) return {kLeftTile, first + j};
  const int at = x * shorts / 8 + j - own;
  return {at < (x + 1) * shorts / 8 ? kShortTile : kNoTile, at};
}

// On the large tile a launch's last round may be cut (forward and transposed-B products).  What an XCD has beyond whole rounds of its 32 units would
// hold them all for a tile's time: up to 8 tiles go out as quarters of 128 x 128, up to 16 as halves of 256 x 128 columns (ffn_piece.h), which
// end 0.25-0.45 and 0.65 of a tile's time later.  Two products of 8 experts, 2048 x 2048: 4096 rows and one expert of 4352 518 us whole, 481 cut; 7
// of them 531 and 503 (nine to sixteen tiles: 4352 rows and one of 4608 531 in whole tiles, 514 in halves; 7 of those 536 and 529, 549 in quarters);
// 1100 rows each 196 and 153, forced onto this tile (tile_of gives them to the half tile, 162); 4096 rows and one 4126, 492 and 481.  From 17 tiles on both forms take as long as the tiles themselves.
// Blocks that find no tile cost a unit 0.38 us each, and after a partial round they run on the units that it leaves idle; after pieces none is idle.
// So launches with more than 2048 of them (imbalanced gates) stay whole: 64 experts, 65536 tokens, Zipf, 1024 x 4096, 8200 blocks for 848 tiles 143 us, 147 cut.
constexpr int kCutQuarters = 8, kCutHalves = 16, kCutSurplus = 2048;
struct TileHalf { int row, col; };          // the half of a tile that a block computes, 0 or 1, or -1: both
// Whether block b may have a part of a tile, in a launch of so many blocks: a test for nearly all of them to fail early.
MOE_HOST_DEVICE inline bool may_be_cut(int b, int blocks, int tiles) { return b / 8 >= ((tiles / 8 - 1) & ~31) && blocks - tiles <= kCutSurplus; }
// What it works on: turns b into the number of the block that would have the whole tile, of which it takes `half`; false where there is nothing for it.
MOE_HOST_DEVICE inline bool cut_tile(int& b, int blocks, int tall, int shorts, TileHalf& half) {
  const int x = b % 8, n = (x + 1) * tall / 8 - x * tall / 8 + (x + 1) * shorts / 8 - x * shorts / 8, over = n % 32, j = b / 8 - (n - over);
  const bool quarters = over <= kCutQuarters;
  const int parts = quarters ? 4 * over : 2 * over;
  if (j < 0 || over > kCutHalves || n - over + parts > blocks / 8) return true;
  if (j >= parts) return false;
  const int low = quarters && j >= 2 * over, k = j - low * 2 * over;           // upper halves first: a short tile has no lower one
  half = {quarters ? low : -1, k % 2};
  b = (n - over + k / 2) * 8 + x;
  return true;
}
// The units of an XCD by when they are free, in twentieths of a whole tile's time.
struct UnitsFree {
  int at[512] = {32}, now = 0, last = 0;
  void take(int n, int time) {                                      // so many tiles or parts, each on the first unit that is free
    while (n > 0) {
      while (at[now] == 0) ++now;
      const int m = n < at[now] ? n : at[now];
      at[now] -= m;
      at[now + time] += m;
      if (now + time > last) last = now + time;
      n -= m;
    }
  }
};
// Whether cut tiles end clearly later than whole ones where every expert's last row tile holds up to 32 rows.  Such a tile takes less than half of a whole one's time, and
// its unit goes on to the next: the whole tiles beyond the full rounds may start long before these end, and their halves, one behind the other on
// the few units that are free early, end later than they would; and halves of such a tile, which both load the rows, take longer than it does.  With a
// multiple of 8 experts every XCD has the same sequence of tiles (apart: the short ones last); this walks it both ways, with what 1300 launches took.  Products whole
// and cut: 16 experts x 516 rows, K = 1536, N = 2048 64.1 and 75.1 us; 8 x 516, 2048 x 3840 80.0 and 89.3; 8 x 1028, 1024 x 4096 92.5 and 100.3; but 32 x 544, 1536 x 1024 82.8 and 70.2.
// Over those launches cutting all is 1.0 % off the better form on average (19 % at most), cutting none 3 %, this 0.4 % (7 % at most where it cuts, 9 % where it does not).
static inline bool cut_short_tiles_end_later(int experts, int row_tiles, int NT, bool apart) {
  constexpr int kTall = 20, kShort = 8, kTallPart[2] = {10, 13}, kShortPart[2] = {6, 11};   // parts: quarters, halves
  const int n = experts * row_tiles * NT, over = n % 32, halves = over > kCutQuarters;
  UnitsFree whole;
  int rest[2 * kCutHalves], runs = 0, done = 0;                     // runs of tiles beyond the full rounds, tall and short in turn
  auto run = [&](int of, bool tall) {
    const int full = n - over - done, early = full > of ? of : (full > 0 ? full : 0);
    done += of;
    whole.take(early, tall ? kTall : kShort);
    if (of == early) return;
    if ((runs % 2 == 0) != tall) rest[runs++] = 0;
    rest[runs++] = of - early;
  };
  if (apart) {
    run(experts * NT * (row_tiles - 1), true);
    run(experts * NT, false);
  } else {
    for (int e = 0; e < experts; ++e)
      for (int c = 0; c < NT; c += 8) {
        const int w = NT - c < 8 ? NT - c : 8;
        run(w * (row_tiles - 1), true);
        run(w, false);
      }
  }
  UnitsFree cut = whole;
  for (int r = 0; r < runs; ++r) {
    whole.take(rest[r], r % 2 == 0 ? kTall : kShort);
    cut.take(2 * rest[r], r % 2 == 0 ? kTallPart[halves] : kShortPart[halves]);
  }
  for (int r = 0; r < runs && !halves; r += 2) cut.take(2 * rest[r], kTallPart[0]);        // lower halves, which short tiles do not have
  return 20 * cut.last >= 21 * whole.last;
}
// Whether a launch gets the kernel that can cut, and the blocks for it: by the tiles of an XCD if every expert has `rows` rows (up to) on average, give or
// take a standard deviation of even choices.  One that has nothing to cut would pay 0.5-1 us for the longer kernel and the blocks (64 experts x 283 rows, 768 x 512:
// second product 25.0 us, 25.9 so); beyond 16 rounds a part of the last one is no more than that either.  The reduction is not asked: 490 drawn products, all experts full or an even
// gate, took 0.83 of the time cut for K = 64, 0.96 for 128 and 256, 0.92 for 384 to 1024 and 0.88 for 1536 and 2048, 240 with a Zipf-shaped gate 0.96, 0.96, 0.90 and 0.92.
static inline bool cuts_last_round(int64_t E, int64_t C, double rows, bool up_to, int64_t NT) {
  const double off = up_to ? sqrt(rows) : 0.0, low = rows - off > 1.0 ? rows - off : 1.0, high = rows + off < (double)C ? rows + off : (double)C;
  const double n = (double)(E * NT) * (ceil(low / kLargeTile) + ceil(high / kLargeTile)) / 16.0;
  if (!(n <= 512.0 && n - 32.0 * floor(n / 32.0) >= 0.5 && n - 32.0 * floor(n / 32.0) <= kCutHalves + 2.0)) return false;
  if (up_to || E % 8 != 0 || C <= kLargeTile || C % kLargeTile == 0 || C % kLargeTile > 32 || (int)n % 32 > kCutHalves) return true;
  const int row_tiles = (int)tiles_in(C, kLargeTile), all = (int)(E * NT) * row_tiles, tall = all - (int)(E * NT);
  if (deals_groups(all, (int)E, (int)NT, 0)) return true;           // another sequence
  return !cut_short_tiles_end_later((int)(E / 8), row_tiles, (int)NT, may_open_a_round(all, 0) && opens_a_round(tall, all, 0));
}

// Which tile block b of a weight-gradient launch (kTN) works on, E experts of MT x NT tiles each; false where there is none for it.
// Hardware deals blocks round-robin: block b runs on XCD b % 8, as the b / 8-th of its tiles.  All experts have the same number of tiles, but a
// tile of an expert with many rows takes several times that of one with few, so every XCD has to get its share of each expert: whole groups of an
// expert's tiles (32 from 1024 tiles on, 16 below, so that they still spread evenly) are dealt
// to the XCDs in turn, then whole tails (what an expert has beyond its groups), and only the groups and tails of the
// last rounds, fewer than eight, are cut into 8 runs of equal length (to a tile).  Runs of an eighth of all tiles gave
// the experts with many rows to one XCD.  Imbalanced gate (Zipf), two products of 8 experts, 8192 tokens, 2048 x 2048: 218 us in groups throughout,
// 417 in eighths, 215 so (training step 800, 986 and 761); 64 experts, 16384 tokens, 1024 x 1024: step 415, 475 and 397.  Even gate, 17 experts x
// 353 rows, 776 x 1544: 81 us in groups throughout, 79 with the tails in eighths, 75 so.
// A launch of one tile to a unit is as long as its slowest tile however it is dealt, and is cut in eighths throughout.  Groups of 8 below 512 tiles
// seldom share a panel: 4 experts, 32895 tokens, 2048 x 768 (384 tiles) step 1186 us, 1169 with 16, 1164 in eighths; imbalanced, 16384, 1024 x 1536
// 355, 347 and 376; 256 tiles, 8192, 1024 x 1024 265 in groups of 8, 258 in eighths.
// No prefix sums over the experts, either, which every tile of a short reduction would pay for.
MOE_HOST_DEVICE inline bool equal_tile(int b, int E, int MT, int NT, TileAt& at) {
  const int n = MT * NT, gs = E * n >= 1024 ? 5 : 4, x = b % 8, i = b / 8;
  const bool deal = E * n > 256;
  const int own = deal ? n >> gs : 0, tail = n - (own << gs), whole = deal ? E >> 3 : 0;        // an expert's groups and what is beyond; rounds of tails
  const int rounds = (E * own) >> 3, dealt = rounds << gs, tails = whole * tail;                // an XCD's
  int e, q;
  if (i < dealt) {
    const int g = (i >> gs) * 8 + x;
    e = g / own;
    q = ((g - e * own) << gs) + (i & ((1 << gs) - 1));
  } else if (i < dealt + tails) {
    const int j = i - dealt, r = j / tail;
    e = r * 8 + x;
    q = (own << gs) + j - r * tail;
  } else {
    const int rest = E * n - 8 * (dealt + tails), t = x * rest / 8 + i - dealt - tails, of_tails = (E - 8 * whole) * tail;
    if (t >= (x + 1) * rest / 8) return false;
    if (t < of_tails) {
      const int r = t / tail;
      e = 8 * whole + r;
      q = (own << gs) + t - r * tail;
    } else {
      const int g = 8 * rounds + ((t - of_tails) >> gs);
      e = g / own;
      q = ((g - e * own) << gs) + ((t - of_tails) & ((1 << gs) - 1));
    }
  }
  at = tile_in_expert(e, q, MT, NT);
  return true;
}

// Row tiles that hold rows, at most, when the experts hold `total` rows among them, each at most C.
static inline int64_t live_row_tiles(int64_t E, int64_t C, int64_t total, int64_t tile_rows) {
  const int64_t full = E * tiles_in(C, tile_rows), n = total / tile_rows + (E < total ? E : total);
  return n < full ? n : full;
}

// Blocks to launch so that every tile is reached whatever the fills turn out to be: of the row tiles of NT tiles each, at most `row_tiles`
// are live in all, and their tiles are dealt evenly to the 8 XCDs (shorts_last: in two kinds, each to a tile).
// The layer knows its total (every choice is one row).  Without it the grid has to hold C rows of every expert, and where the
// capacity is far above the mean fill nearly all blocks find nothing to do, each after a tile search and holding its LDS: dynamic
// capacity, buffers for all 2048 tokens, 128 experts, M = 4096, H = 1024: layer 746 us, 487 with the bound.
static inline int64_t tile_grid(int64_t NT, int64_t row_tiles, bool shorts_last = false, bool cuts = false) {
  return (tiles_in(row_tiles * NT, 8) + (shorts_last ? 1 : 0) + (cuts ? 3 * kCutQuarters : 0)) * 8;
}

// Shapes the 256 x 256 tile takes in the forward layout; gather_rows > 0: A's rows are gathered from that many.
static inline bool large_tile_supports(int64_t E, int64_t C, int64_t K, int64_t N, int64_t gather_rows) {
  if (K % kLargeK != 0 || N % kLargeTile != 0 || E > kMaxExperts) return false;
  const int64_t tiles = E * tiles_in(C, kLargeTile) * (N / kLargeTile);
  // 32-bit byte offsets inside one expert's A slab and B matrix; in a gathered matrix offsets may count 16-byte pieces
  const int64_t a_rows = gather_rows > 0 ? gather_rows : C, a_bytes = (int64_t)1 << (gather_rows > 0 ? 36 : 32);
  return tiles < ((int64_t)1 << 30) && a_rows * K * 2 < a_bytes && K * N * 2 < ((int64_t)1 << 32) && gather_rows < ((int64_t)1 << 31);
}

// Whether byte offsets into a gathered matrix of rows of K bf16 values need more than 32 bits.
static inline bool far_rows(int64_t gather_rows, int64_t K) { return gather_rows * K * 2 >= ((int64_t)1 << 32); }

// Shapes for which the three layouts of an expert layer's backward run on it.
static inline bool large_tile_supports_backward(int64_t E, int64_t C, int64_t M, int64_t H) {
  const int64_t W = M > H ? M : H;
  const int64_t tiles = E * tiles_in(C > W ? C : W, kLargeTile) * (W / kLargeTile);
  return M % kLargeTile == 0 && H % kLargeTile == 0 && E <= kMaxExperts && tiles < ((int64_t)1 << 30) &&
         C * W * 2 < ((int64_t)1 << 32) && M * H * 2 < ((int64_t)1 << 32);
}

// Which tile a bf16 launch takes: the one with the least estimated time among those it may run on (tile_of), in microseconds
//   base + fix * rounds + ksteps * max(lat * rounds, thr * tiles per unit),    rounds = tiles per unit / blocks per unit
// but for few rows of large weights (streamed tiles, below).  The shapes differ in how much of the chip a launch of few tiles uses, how finely
// its work divides among the 256 compute units, and how fast a full unit runs: 256 x 256 (one block per unit) was 1.2-1.3 times as
// fast as 128 x 128 (two) with the kernel that the constants were fitted on, and is 1.7-1.9 times as fast as 64 x 64 (three) once every unit has several tiles, and the slowest by up to
// 3 times where it leaves most units idle.  128 x 256 (kHalf, two blocks, ffn_half.h) costs more per product than 256 x 256 and less per tile.
//
// The constants were fitted to launches by themselves, with a 128 x 128 kernel of 32 x 32 x 16 instructions (the present one takes 0.82 to 0.99 of
// its time, by layout: ffn_ring.h) and tiles numbered in groups throughout, and so are all distances and times of this comment: with
// the kernels as they are they have not been taken again.  Over launches drawn from 4-128 experts, 50-4200
// rows each, K and N 256-4096, the choice was off the best tile by, on average: 3.2 % in 315 forward products (gathered with GELU, and
// plain; 34 % for always the large tile), 4.1 % in 75 that keep their pre-activations (43 %), 2.8 and 5.3 % in 85 with B transposed, plain
// and times act' (24, 30 %), 2.5 % in 205 weight gradients of slabs (28 %), 0.9 % in 205 gathered ones (9 %).  Products that follow each
// other run at the board's power limit and take 1.2-1.7 times the estimate on the large tile; the choice holds in whole layers all the same.
//   256 x 256: thr 1.1.  0.98, which its main loop reaches, took products from tiles that run them faster: 100 of those between the two
//     with B transposed at 1.07 times their time (median, up to 1.6), 130 that keep their pre-activations at 1.28, 350 weight
//     gradients of slabs at 1.21 (17 experts x 292 rows, 2560 x 1024: 55.7 and 41.4 us).  Gathered weight gradients have 0.98: of the same
//     350 the large tile is the faster of nearly all (0.91; 52.4 and 56.7 us), and 0.98 chooses 0.8 % off the better, 1.1 11.6 %.
//   128 x 256: a block that has its unit for itself takes 1.2 us per K-step of 64 (its ring holds 48 KB ahead), two together 1.6.  Over 1145
//     forward products these constants choose 3.6 % off the best, 60 of them over 4 % slower than without this tile (1.29 at most) and
//     292 as much faster (3.1 %, 33 and 259 over 940 drawn afterwards); with lat 0.33, thr 0.72 and margins instead it was 5.8 %, 137
//     slower (up to 1.64: 48 experts x 190 rows, 4096 x 512, 105 us here and 67 on 128 x 128) and 329 faster.  Rows that a 64-row tile holds never come here: half of the tile
//     would be padding.  (Over 79 such products it would choose 5.2 % off the best instead of 6.5 %, but take up to 1.19 times their
//     time: 96 experts x 53 rows, 2560 x 1280, 157 us here and 132 on 64 x 128.)
//     Two products, on the large tile and here: 8 experts x 1100 rows, 2048 x 2048 181 and 165 us; 8 x 2048 239 and 268; 32 x 784, 768 x
//     3072 327 and 315, with 784 rows on average 335 and 349 (whole ViT passes 390 and 385, 634 and 635).
//     Forward products only: with a transposed B (64-byte pieces of k, where the large tile loads 128) it is the slower at nearly
//     every size (backward of 32 x 784 rows: 251 and 198 us against 226 and 171), and a training step's first product, which
//     writes twice, gains nothing (216 against 212).
// Where the large tile's last round is cut (cuts_last_round), the estimate still counts a whole one: what it says of such launches is too much.
//   64 x 128 (two blocks) is for the launches between: two products of 8 experts x 96 rows, K = N = 2048: 68 us on 128 x 128 and 61
//     on 64 x 64 -> 53.
//
// Experts of so few rows that one tile holds them read their weights once, and that is all their launch does: 64 x 128 with the
// nontemporal hint on the weights, 64 experts x 16 rows, 1024 x 4096, two products 221 -> 189 us (5.2 -> 6.1 TB/s over both; the
// hint alone 202).  Where that leaves units without a block, 64 x 64 one stage deeper (8 experts x 16 rows, 2048 x 2048: 40 -> 33 us).
// Weights below 48 MB keep the plain loads: they may stay in the caches from one call to the next (17 experts, 776 x 1544,
// 32 rows: 39 us plain, 41 streamed).
enum class Tile { k256, k128, k64x128, k64, k64x128_stream, k64_stream, kHalf };

static inline double tile_cost(Tile tile, int mode, int64_t E, int64_t rows, double mean_rows, int64_t K, int64_t N, bool gathered) {
  const double ksteps = (mode == kTN ? mean_rows : (double)K) / 64 + 0.5;
  auto cost = [&](int bm, int bn, int per_unit, double base, double fix, double lat, double thr) {
    // an average fill ends in half a tile, but no expert has more row tiles than its slab (without this bound 24 experts x 256
    // rows, 2048 x 2048, counted as 1.5 tiles each: two products 180 us on smaller tiles, 137 on the large one)
    const double full = (double)tiles_in(rows, bm), some = mean_rows / bm + 0.5;
    const double row_tiles = mode == kTN || some > full ? full : (some > 1.0 ? some : 1.0);
    double q = (double)E * row_tiles * (double)tiles_in(N, bn) / 256.0;             // tiles per compute unit
    q = q <= 4.0 * per_unit ? ceil(q - 0.02) : q + 0.5;
    const double rounds = q > per_unit ? q / per_unit : 1.0;
    return base + fix * rounds + ksteps * (lat * rounds > thr * q ? lat * rounds : thr * q);
  };
  switch (tile) {
    // kTN: with the launch that pads its last K-step, and, where its rows are gathered, less (see above)
    case Tile::k256: return cost(256, 256, 1, mode == kTN ? 10.0 : 1.0, 9.0, 0.0, mode == kTN && gathered ? 0.98 : 1.1);
    case Tile::kHalf: return cost(128, 256, 2, 2.0, 3.0, 1.2, 0.8);
    case Tile::k64x128: return cost(64, 128, 2, 2.5, 2.5, 0.3, 0.44);
    case Tile::k64: return cost(64, 64, 3, 3.0, 1.5, 0.3, 0.235);
    default: return cost(128, 128, 2, 1.5, 3.5, 0.3, 0.56);
  }
}

// large_ok, half_ok: whether the launch may run on the large tile, and on its half.
static inline Tile choose_tile(int mode, bool large_ok, bool half_ok, int64_t E, int64_t rows, double mean_rows, int64_t K, int64_t N, bool gathered) {
  if (mode != kTN && mean_rows <= 48.0 && (double)E * K * N * 2 >= 48e6) return E * tiles_in(N, 128) >= 256 ? Tile::k64x128_stream : Tile::k64_stream;
  auto estimate = [&](Tile t) { return tile_cost(t, mode, E, rows, mean_rows, K, N, gathered); };
  Tile best = Tile::k128;
  double least = estimate(best);
  auto consider = [&](Tile t) {
    const double c = estimate(t);
    if (c < least) { least = c; best = t; }
  };
  if (large_ok) consider(Tile::k256);
  if (large_ok && half_ok && mean_rows > 64.0) consider(Tile::kHalf);
  if (mode != kTN) {                                                // 64 x 64 was the best tile for one of 278 weight gradients
    consider(Tile::k64x128);
    consider(Tile::k64);
  }
  return best;
}

// fp32 products (forward layout or B transposed) whose 32 x 32 tiles are all on the chip at once, two blocks to a unit, split each
// tile's reduction over four waves.  On 64 x 64 such a launch is one chain of fp32 matrix instructions per wave on a part of the units.  Two
// products: 4 experts x 256 rows, 256 x 512 (512 and 256 tiles): 22.0 -> 15.4 us; 8 x 32, 1024 x 2048: 61 -> 34; 8 x 16, 2048 x 2048: 81 -> 56.
// With a second round of blocks 64 x 64, which loads half as much per product, is the faster: 4 x 512, 256 x 512 (1024 and 512 tiles):
// 23.5 there, 25.0 here; 8 x 512: 28.5 and 44.9.  Up to 64 k, which is two K-steps for four waves, 64 x 64 is the faster, too: 4 x 256 rows,
// N = 512: K = 32 4.8 us there, 5.5 here, 64 5.5 and 5.9, 96 6.0 and 6.0, 128 6.5 and 6.3, 256 8.6 and 7.7.  Only the sizes of the buffers
// decide, so that every route to a product sums alike.
constexpr int kSplitTile = 32, kSplitParts = 4;
static inline bool fp32_split(int64_t E, int64_t C, int64_t K, int64_t N) { return K > 64 && E * tiles_in(C, kSplitTile) * tiles_in(N, kSplitTile) <= 512; }

// Rows an expert holds on average: the caller's hint, or all of them.
static inline double mean_or(int64_t rows_hint, int64_t C) { return (double)(rows_hint > 0 && rows_hint < C ? rows_hint : C); }

// The tile of a bf16 product: out[e] (C x N) over K, with A gathered from gather_rows rows where that is > 0 (kNN); over the slots K
// of an expert, of which rows_hint are filled on average, for an output of C x N (kTN).  keeps_pre (kNN): the values before the
// activation are written as well.  The half tile writes one result and takes 32-bit offsets only.
static inline Tile tile_of(int mode, int64_t E, int64_t C, int64_t K, int64_t N, int64_t rows_hint, int64_t gather_rows, bool keeps_pre) {
  if (mode == kTN)
    return choose_tile(kTN, large_tile_supports_backward(E, K, C, N) && gather_rows * C * 2 < ((int64_t)1 << 36), false, E, C, mean_or(rows_hint, K), K, N,
                       gather_rows > 0);
  const bool large_ok = large_tile_supports(E, C, K, N, mode == kNN ? gather_rows : 0);
  const bool half_ok = mode == kNN && !keeps_pre && !far_rows(gather_rows, K);
  return choose_tile(mode, large_ok, half_ok, E, C, mean_or(rows_hint, C), K, N, gather_rows > 0);
}

// Whether the column sums (ffn_backward.hip) of E slabs each, of so many rows on average and of the given bytes (0: not summed), are streamed, in
// pieces of 256 bytes to a row instead of 128: where the rows that are expected lie far beyond the caches and half as many blocks still fill the chip.
// Without and with, both sums: 128 experts x 2048 rows, 4096 and 1024 columns 537 and 475 us; 64 x 4096, 2048 and 2048 416 and 330; fewer blocks than
// units: 8 x 16384, 1024 and 1024 (128) 103 and 108, 4 x 32768, 1024 and 1024 (64) 141 and 185, 5 x 78643, 256 and 256 (10) 244 and 371.  The
// capacity says little: of 64 x 2560, 1024 and 1024, a Zipf-shaped gate fills 77 MB, which the caches hold, 12.9 and 16.0.  With an even
// gate the line could lie at 256 MB (8 x 4096, 2048 and 2048 54 and 44; 134 MB of 8 x 4096, 1024 and 1024 22.5 and 23.0).
static inline bool colsum_streams(int64_t E, double rows, int64_t row_bytes1, int64_t row_bytes2) {
  return (double)E * rows * (double)(row_bytes1 + row_bytes2) >= 1073741824.0 && E * (tiles_in(row_bytes1, 256) + tiles_in(row_bytes2, 256)) >= 256;
}

}  // namespace moe
