"""The host rules of the grouped GEMM and of the gate (csrc/ffn_rules.h, csrc/gate_rules.h), compiled on their own: no GPU needed."""
import ctypes

import numpy as np
import pytest


def blocks_needed(tiles, NT):
    """Blocks the kernels' tile search can ask for when expert e has tiles[e] live row tiles of NT tiles each: as many for each of 8 XCDs."""
    return -(-int(tiles.sum()) * NT // 8) * 8


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("seed", range(8))
def test_grid_reaches_every_tile(ffn_rules, seed, half):
    """Whatever the fills are, as long as they keep to the total the caller promises, in all and expert by expert."""
    rng = np.random.default_rng(seed)
    for _ in range(3000):
        E, tile = int(rng.integers(1, 513)), int(rng.choice([64, 128, 256])) if not half else 128
        C, NT = int(2 ** rng.uniform(0, 14)), int(2 ** rng.uniform(0, 7))
        total = int(rng.integers(1, E * C + 1)) if rng.random() < 0.5 else E * int(rng.integers(1, C + 1))
        kind = rng.integers(4)
        if kind == 0:                                  # as many experts with one row over a whole tile as the total allows
            fills = np.full(E, min(C, int(rng.integers(0, C // tile + 1)) * tile + 1))
        elif kind == 1:                                # one row each, the rest to a few
            fills = np.ones(E, dtype=np.int64)
            fills[:max(1, E // 16)] = C
        elif kind == 2:
            fills = np.minimum(rng.multinomial(total, rng.dirichlet(np.full(E, 0.2))), C)
        else:
            fills = rng.integers(0, C + 1, size=E)
        fills = np.minimum(fills, np.maximum(total - (np.cumsum(fills) - fills), 0))      # within the total
        assert fills.sum() <= total
        grid = ffn_rules.grid(E, C, tile, NT, total, 0)
        assert grid >= blocks_needed(-(-fills // tile), NT), (E, C, tile, NT, total)


def test_grid_is_bounded_by_the_rows_that_exist(ffn_rules):
    """Buffers sized for every token, 128 experts: the grid follows the 4096 rows that exist, not 128 x 2048."""
    E, T, k = 128, 2048, 2
    for tile, NT in ((64, 8), (64, 32), (128, 16), (256, 4)):
        live = (T * k // tile + E) * NT
        assert ffn_rules.grid(E, T, tile, NT, T * k, 0) <= live + 7
        assert E * T // tile * NT <= ffn_rules.grid(E, T, tile, NT, E * T, 0) <= E * T // tile * NT + 7


def tiles_of_xcds(find, blocks):
    """What find(b), a tile or None, gives for blocks 0 .. blocks - 1, XCD by XCD; none past them."""
    assert all(find(b) is None for b in range(blocks, blocks + 64))
    return [[t for t in (find(b) for b in range(x, blocks, 8)) if t is not None] for x in range(8)]


def equal_tiles(ffn_rules, E, MT, NT):
    at = (ctypes.c_int * 3)()
    find = lambda b: tuple(at) if ffn_rules.equal_tile(b, E, MT, NT, at) else None
    return tiles_of_xcds(find, -(-E * MT * NT // 8) * 8)


@pytest.mark.parametrize("E", [1, 3, 7, 8, 9, 17, 64, 65, 512])
def test_weight_gradient_tiles_once(ffn_rules, E):
    """Every tile of a weight-gradient launch has one block, below and beyond each group size, and no XCD a tile more than another but for one."""
    for MT, NT in [(1, 1), (1, 7), (2, 8), (3, 4), (5, 9), (8, 8), (7, 13), (19, 16)]:
        if E * MT * NT > 40000:
            continue
        per = equal_tiles(ffn_rules, E, MT, NT)
        assert sorted(sum(per, [])) == [(e, m, n) for e in range(E) for m in range(MT) for n in range(NT)]
        assert max(map(len, per)) - min(map(len, per)) <= 1


@pytest.mark.parametrize("E,MT,NT", [(8, 8, 8), (8, 6, 8), (16, 4, 16), (32, 12, 4), (32, 3, 12), (64, 4, 4), (64, 8, 16)])
def test_weight_gradient_work_is_even_on_imbalanced_experts(ffn_rules, E, MT, NT):
    """A Zipf-shaped gate: the first experts are full, the last nearly empty.  A tile costs its reduction (up to 32 K-steps) and a fixed
    part of 8.  No XCD has more than 1.25 times the mean (runs of an eighth of the tiles: more than twice)."""
    cost = [8 + min(32, max(1, round(64 / (e * 8 / E + 1) ** 1.5))) for e in range(E)]
    per = [sum(cost[t[0]] for t in x) for x in equal_tiles(ffn_rules, E, MT, NT)]
    assert max(per) <= 1.25 * sum(per) / 8
    order = sorted((e, m, n) for e in range(E) for m in range(MT) for n in range(NT))
    eighths = [sum(cost[t[0]] for t in order[x * len(order) // 8:(x + 1) * len(order) // 8]) for x in range(8)]
    assert max(eighths) > 1.5 * sum(eighths) / 8


def live_tiles(ffn_rules, rows, tile_rows, NT, shift, blocks, parts=None, shorts_last=0):
    """The tiles of a forward launch, XCD by XCD; `parts` gets what kinds of place in the numbering they came from."""
    at, fills = (ctypes.c_int * 3)(), (ctypes.c_int * len(rows))(*rows)
    def find(b):
        part = ffn_rules.tile_at(b, len(rows), fills, tile_rows, NT, shift, shorts_last, at)
        assert part >= 0
        if parts is not None and part:
            parts.add(part)
        return tuple(at) if part else None
    return tiles_of_xcds(find, blocks)


@pytest.mark.parametrize("shift,shorts_last", [(0, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("E,C,tile_rows,NT,most_dealt", [(1, 700, 64, 3, -1), (8, 4200, 256, 8, 0), (17, 353, 128, 14, -1), (33, 1500, 128, 9, 1), (70, 1300, 128, 12, 1),
                                                         (130, 900, 64, 5, 1), (65, 66, 64, 9, -1), (512, 300, 64, 7, 0)])
def test_every_live_tile_once(ffn_rules, E, C, tile_rows, NT, most_dealt, shift, shorts_last):
    """Fills of every kind, in launches below and beyond the tiles from which whole groups are dealt: every live tile has one block
    among those that the grid launches, and no XCD has a tile more than another but for one of each kind.  most_dealt: the largest shift at which groups are."""
    rng, parts = np.random.default_rng(E), set()
    for fills in (np.full(E, C), rng.integers(0, C + 1, size=E), np.where(rng.random(E) < 0.3, C, 0), np.minimum(C, (C * 4 / (1 + np.arange(E))).astype(int)),
                  np.minimum(C, np.array([0, 1, tile_rows, tile_rows + 1, 2 * tile_rows, C, C - 1])[rng.integers(0, 7, size=E)])):
        rows = [int(v) for v in fills]
        grid = ffn_rules.grid(E, C, tile_rows, NT, max(1, sum(rows)), shorts_last)
        per = live_tiles(ffn_rules, rows, tile_rows, NT, shift, grid, parts, shorts_last)
        assert sorted(sum(per, [])) == [(e, m, n) for e in range(E) for m in range(-(-rows[e] // tile_rows)) for n in range(NT)]
        assert max(map(len, per)) - min(map(len, per)) <= 1 + shorts_last
    assert 2 in parts and (1 in parts) == (shift <= most_dealt) and (3 in parts) == (shorts_last == 1 and E > 1)


@pytest.mark.parametrize("E,C,tile_rows,NT,worse", [(64, 550, 256, 4, 1.2), (8, 3000, 256, 8, 1.05), (32, 980, 128, 12, 1.15), (128, 586, 128, 8, 1.15)])
def test_short_row_tiles_are_shared_evenly(ffn_rules, E, C, tile_rows, NT, worse):
    """Zipf-shaped fills: a tile costs a third and, for the rest, its rows.  No XCD has more than 1.15 times the mean; with one run for all kinds
    of tiles it is at least `worse` times as much."""
    fills = [max(1, min(C, int(C * (E / 2) * (e + 1) ** -2.4))) if e < E // 2 else 30 for e in range(E)]
    def most(shorts_last):
        blocks = ffn_rules.grid(E, C, tile_rows, NT, sum(fills), shorts_last)
        work = [sum(0.35 + 0.65 * min(1, (fills[e] - m * tile_rows) / tile_rows) for e, m, _ in x)
                for x in live_tiles(ffn_rules, fills, tile_rows, NT, tile_rows == 128, blocks, shorts_last=shorts_last)]
        return max(work) * 8 / sum(work)
    assert most(1) <= 1.15 and most(0) >= worse * most(1)


def test_an_even_gate_keeps_short_row_tiles_in_place(ffn_rules):
    """Fills as an even gate gives them, from 30 rows per expert on: no expert is far above the mean, so the shorts stay with the others.  They come
    last where they alone open the second or third round of the chip and are few."""
    rng, parts = np.random.default_rng(1), set()
    for E, mean in [(8, 4096), (32, 784), (17, 353), (64, 128), (128, 64), (32, 30)]:
        rows = [int(v) for v in rng.multinomial(E * mean, np.full(E, 1 / E))]
        live_tiles(ffn_rules, rows, 128, 6, 1, ffn_rules.grid(E, 2 * mean, 128, 6, E * mean, 1), parts, 1)
    assert 3 not in parts
    for E, mean, tile_rows, NT, apart in [(32, 500, 256, 8, True), (32, 256, 128, 8, True), (64, 166, 128, 8, False), (32, 450, 256, 8, False), (32, 1000, 256, 8, False)]:
        rows, parts = [mean + (16 if e % 4 == 0 else -16) for e in range(E)], set()
        per = live_tiles(ffn_rules, rows, tile_rows, NT, int(tile_rows == 128), ffn_rules.grid(E, 2 * mean, tile_rows, NT, sum(rows), 1), parts, 1)
        assert sorted(sum(per, [])) == [(e, m, n) for e in range(E) for m in range(-(-rows[e] // tile_rows)) for n in range(NT)]
        assert (3 in parts) == apart, (E, mean)


def panels(tiles, at_once):
    """Panels of A and B (256 columns of B as 2 of 128 rows of A) that an XCD brings into its L2, as many tiles at a time as it holds."""
    return sum(len({t[:2] for t in w}) + 2 * len({(t[0], t[2]) for t in w}) for w in (tiles[i:i + at_once] for i in range(0, len(tiles), at_once)))


@pytest.mark.parametrize("E,rows,NT,in32", [(32, 784, 12, 1.35), (32, 2000, 8, 1.6), (16, 4000, 8, 1.6), (64, 1000, 10, 1.1), (128, 470, 8, 1.0), (8, 8000, 4, 1.0)])
def test_groups_of_the_half_tile_are_what_an_xcd_holds(ffn_rules, E, rows, NT, in32):
    """Two blocks of the half tile share a unit, so an XCD holds 64 of its tiles at one time.  At most 1.1 times the panels of groups of
    64 dealt one by one, short ones last; with groups of 32 it is in32 times and more."""
    MT = -(-rows // 128)
    order = [[(e, m, 8 * c + n) for c in range(-(-NT // 8)) for m in range(MT) for n in range(min(8, NT - 8 * c))] for e in range(E)]
    cut = [t[i:i + 64] for t in order for i in range(0, len(t), 64)]
    groups = [g for g in cut if len(g) == 64] + [g for g in cut if len(g) < 64]
    old = sum(panels(sum(groups[x::8], []), 64) for x in range(8))
    now = sum(panels(x, 64) for x in live_tiles(ffn_rules, [rows] * E, 128, NT, ffn_rules.half_shift(), -(-E * MT * NT // 8) * 8))
    assert now <= 1.1 * old
    assert sum(panels(x, 64) for x in live_tiles(ffn_rules, [rows] * E, 128, NT, 0, -(-E * MT * NT // 8) * 8)) >= in32 * old


def test_column_sums_stream_what_is_expected_and_summed(ffn_rules):
    """The rows expected, not the capacity, of the slabs whose sum is asked for, and only with a block for every unit."""
    big = dict(E=128, M=8192, H=2048)                                # bytes of a row, 2048 rows expected of 4096
    assert ffn_rules.colsum_streams(big["E"], 2048, big["H"], big["M"])
    assert not ffn_rules.colsum_streams(big["E"], 200, big["H"], big["M"])       # the same buffers, mostly empty
    assert not ffn_rules.colsum_streams(big["E"], 2048, big["H"], 0)             # the wide slab's sum is not asked for
    assert not ffn_rules.colsum_streams(4, 131072, 2048, 2048)                   # 64 blocks


K256, K128, K64X128, K64, K64X128_STREAM, K64_STREAM, KHALF = range(7)


@pytest.mark.parametrize("seed", range(4))
def test_half_tile_only_where_it_may_run(ffn_rules, seed):
    """A product that keeps its pre-activations, or gathers from 4 GiB and more, runs on the whole large tile or on a smaller one: the
    estimate of the half must not speak for the whole (48 experts x 96 rows, 256 x 3072: 41 us estimated, 23 on the 128 x 128 tile)."""
    rng = np.random.default_rng(seed)
    products = [(48, 96, 256, 3072, 0), (48, 320, 256, 1024, 256), (17, 96, 2048, 4096, 0), (128, 128, 4096, 768, 0)]
    for _ in range(3000):
        E, C = int(2 ** rng.uniform(2, 7)), int(2 ** rng.uniform(6, 13))
        products.append((E, C, 64 * int(rng.integers(4, 65)), 256 * int(rng.integers(1, 17)), int(rng.integers(C // 4, C + 1))))
    other = 0
    for E, C, K, N, hint in products:
        far = 2 ** 32 // (2 * K) + 1
        if ffn_rules.tile(0, E, C, K, N, hint, 0) == KHALF:
            other += 1
        for tile in (ffn_rules.tile_keeping_pre(E, C, K, N, hint, 0), ffn_rules.tile(0, E, C, K, N, hint, far)):
            assert tile != KHALF
            if tile not in (K64X128_STREAM, K64_STREAM):
                cost = [ffn_rules.tile_cost(t, 0, E, C, K, N, hint, 0) for t in (K256, K128, K64X128, K64)]
                assert cost[tile] == min(cost), (E, C, K, N, hint)
    assert other > 100                                 # products that do run on the half without either


def test_half_tile_not_alone_on_its_unit(ffn_rules):
    """Products of few tiles, whose blocks have a unit each for themselves, run longer on the half tile than on a smaller one
    (microseconds: there, here); rows that a 64-row tile holds never take it; those it is for do."""
    for E, C, mean, K, N in ((48, 190, 190, 4096, 512),          # 67, 105
                             (24, 105, 105, 2560, 1536),         # 42, 62
                             (32, 144, 115, 2048, 1024),         # 38, 52
                             (20, 178, 89, 3072, 2560),          # 73, 115
                             (12, 118, 59, 3072, 4096), (128, 128, 64, 3072, 2048), (96, 64, 64, 1280, 3072)):
        assert ffn_rules.tile(0, E, C, K, N, mean, 0) != KHALF, (E, C, K, N)
    for E, C, mean, K, N in ((32, 980, 784, 768, 3072), (32, 980, 784, 3072, 768), (8, 1100, 1100, 2048, 2048), (8, 21056, 21056, 512, 256)):
        assert ffn_rules.tile(0, E, C, K, N, mean, 0) == KHALF, (E, C, K, N)


def test_tile_of_transposed_operands(ffn_rules):
    """Products with B transposed, and weight gradients of dispatched slabs, that a smaller tile runs faster (second figure) than the
    large one (first); the same weight gradients with gathered rows, which are the faster on the large one."""
    for E, C, mean, K, N in ((20, 5348, 1337, 3072, 256),        # 70.0, 61.2 us
                             (6, 868, 217, 4096, 4096),          # 85.8, 72.9
                             (24, 105, 105, 2560, 1536)):        # 54.7, 44.4
        assert ffn_rules.tile(1, E, C, K, N, mean, 0) != K256, (E, C, K, N)
    for E, C, mean, R, N in ((17, 292, 292, 2560, 1024),         # 55.7, 41.4; gathered 52.4, 56.7
                             (24, 3106, 1553, 1536, 512),        # 87.0, 74.5; 91.8, 107.4
                             (8, 1008, 806, 1024, 3072)):        # 58.0, 47.6; 59.0, 62.8
        assert ffn_rules.tile(2, E, R, C, N, mean, 0) == K128, (E, C, R, N)
        assert ffn_rules.tile(2, E, R, C, N, mean, E * mean) == K256, (E, C, R, N)


def test_tile_of_exact_row_counts(ffn_rules):
    """Slabs whose rows fill whole row tiles of 256, or stay short of one: the large tile or its half, which measured 13 to 32 % faster there
    than what a row count taken for an average one chose (32 experts x 160 rows, 2048 x 2048: 146 against 176 us)."""
    for E, C, M, H in ((24, 224, 2048, 2048), (24, 256, 2048, 2048), (32, 160, 2048, 2048), (32, 192, 2048, 2048), (16, 448, 2048, 2048),
                       (64, 192, 1024, 4096), (32, 448, 4096, 1024), (32, 448, 1024, 4096)):
        assert ffn_rules.tile(0, E, C, M, H, 0, 0) in (K256, KHALF) and ffn_rules.tile(0, E, C, H, M, 0, 0) in (K256, KHALF), (E, C, M, H)


def test_tile_of_tokens_beyond_4_gib(ffn_rules):
    """Rows gathered from a token matrix of 4 GiB and more stay on the large tile, forward and in the weight gradient (on the
    128 x 128 tile a layer of 2^19 tokens, M = H = 4096, took 35.8 ms instead of 32.3)."""
    T, M, H, E = 2 ** 19, 4096, 4096, 8
    assert ffn_rules.tile(0, E, T // E, M, H, T // E, T) == K256
    assert ffn_rules.tile(2, E, M, T // E, H, T // E, T) == K256
    assert ffn_rules.tile(0, E, T // E, M, H, T // E, 2 ** 23) != K256       # 64 GiB: beyond the kernel's offsets


def test_fp32_split_where_it_is_the_faster(ffn_rules):
    """The split 32 x 32 tile only for reductions of three K-steps and more (4 experts x 256 rows, N = 512: K = 32 4.8 us without and 5.5
    with it, 64 5.5 and 5.9, 128 6.5 and 6.3), and only where all its tiles are on the chip at once."""
    for K in (8, 32, 64, 72, 96, 512):
        assert ffn_rules.split(4, 256, K, 512) == (K > 64) and not ffn_rules.split(4, 257, K, 512)


def test_slots_in_one_launch_where_it_is_the_faster(ffn_rules):
    """Scan and assignment in one launch only where that measured faster than two (both sides beside the rule)."""
    for T, E, k in ((64, 8, 2), (2048, 8, 2), (8192, 8, 1), (4096, 8, 2), (1024, 32, 2), (512, 64, 2), (64, 16, 4)):
        assert ffn_rules.one_launch(T, E, k), (T, E, k)
    for T, E, k in ((16384, 8, 1), (32768, 8, 1), (16384, 8, 2), (8192, 8, 4), (4096, 16, 2), (8192, 32, 1), (64, 32, 1), (64, 64, 2),
                    (256, 64, 4), (256, 128, 1)):
        assert not ffn_rules.one_launch(T, E, k), (T, E, k)


def test_gate_dx_tokens_per_block(ffn_rules):
    """Sixteen tokens to a block wherever four had measured slower than before (fp32 rows of M x 4 bytes, bf16 of M x 2)."""
    for T, row_bytes in ((1024, 8192), (2048, 8192), (4096, 8192), (1024, 16384), (2048, 16384), (4096, 3104), (8192, 1024), (8192, 4096)):
        assert ffn_rules.dx_tokens(T, row_bytes) == 16, (T, row_bytes)
    for T, row_bytes in ((64, 1024), (1024, 1024), (4096, 1024), (1024, 3104), (256, 8192), (256, 16384), (3001, 1552), (1024, 4096)):
        assert ffn_rules.dx_tokens(T, row_bytes) == 4, (T, row_bytes)


def test_gate_backward_tokens_per_block(ffn_rules):
    """One round per block wherever its rounds had measured slower than before; never 2^24 blocks of 256 threads."""
    for T, E in ((8192, 4), (16384, 4), (32768, 8), (16384, 16), (65535, 8)):
        assert ffn_rules.backward_tokens(T, E, 0) == (32 if E <= 8 else 16), (T, E)
    assert ffn_rules.backward_tokens(65536, 4, 0) == 64 and ffn_rules.backward_tokens(16384, 8, 1) == 64
    for T in (2 ** 28, 2 ** 29, 2 ** 30 - 63, 2 ** 30):
        for E in (1, 8, 9, 128, 129, 512):
            for bias in (0, 1):
                assert -(-T // ffn_rules.backward_tokens(T, E, bias)) < 2 ** 24


def test_wide_logits(ffn_rules):
    """Whole 128s of experts where they measured faster than 64 at a time on the narrow kernel, and never a remainder that would mostly be padding."""
    for T, E, wide in ((65536, 128, 128), (65536, 136, 128), (65536, 120, 120), (65536, 96, 0), (65536, 65, 0), (65536, 192, 128), (12000, 512, 512),
                       (8200, 136, 0), (16384, 128, 0), (25088, 256, 256), (65536, 64, 0)):
        assert ffn_rules.wide_logits(T, E, 1) == wide, (T, E)
    assert ffn_rules.wide_logits(65536, 129, 0) == 0


def test_lane_topk_line(ffn_rules):
    """512 blocks of 64 tokens for few choices and without repairs; with repairs further out the longer their products, sooner for few experts."""
    line = ffn_rules.lane_topk_blocks
    assert {line(E, k, M) for E in (17, 64, 128, 512) for k, M in ((1, 4096), (4, 4096), (5, 0), (32, 0))} == {512}
    assert line(32, 8, 1024) == 512 and line(128, 8, 4096) == 1024
    for E, k in ((32, 5), (64, 8), (512, 16)):
        lines = [line(E, k, M) for M in range(256, 16384, 256)]
        assert lines == sorted(lines) and lines[0] == 512 and lines[-1] == 1024
        assert line(32, k, 2048) <= line(64, k, 2048)
