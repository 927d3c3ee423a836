"""The parts of tiles that the large tile's last round is cut into (cut_tile in csrc/ffn_rules.h, csrc/ffn_piece.h)."""
import ctypes
import heapq
import itertools
import os
import subprocess

import numpy as np
import pytest
import torch

from oracle import moe_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SOURCE = r"""
#include "paper_2206_03382_amd/csrc/ffn_rules.h"
extern "C" {
int64_t grid(int64_t tiles) { return moe::tile_grid(1, tiles, true, true); }
int cuts(int64_t E, int64_t C, double rows, int up_to, int64_t NT) { return moe::cuts_last_round(E, C, rows, up_to, NT); }
// as the kernel's search does it: the block whose tile block b works on, row and column half; false where there is nothing for b
int part(int b, int blocks, int tall, int shorts, int rounds, int* at) {
  moe::TileHalf half = {-1, -1};
  if (moe::may_be_cut(b, blocks, tall + shorts) && !moe::cut_tile(b, blocks, tall, shorts, half)) return 0;
  at[0] = b; at[1] = half.row; at[2] = half.col; at[3] = moe::tile_spot(b, tall, shorts, rounds, moe::kGroupShift).part == moe::kDealtTile;
  return moe::tile_spot(b, tall, shorts, rounds, moe::kGroupShift).part != moe::kNoTile;
}
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("cuts")
    (d / "cuts.cpp").write_text(SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", ROOT, str(d / "cuts.cpp"), "-o", str(d / "cuts.so")], check=True)
    lib = ctypes.CDLL(str(d / "cuts.so"))
    lib.grid.restype, lib.grid.argtypes = ctypes.c_int64, [ctypes.c_int64]
    lib.cuts.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_double, ctypes.c_int, ctypes.c_int64]
    return lib


def test_every_quarter_of_every_tile_once(rules):
    """Any number of tall and short tiles, with any number of whole groups dealt first, in a grid for just those and in one with room: every tile is computed
    whole or in all its parts, once, and those of dealt groups whole."""
    rng, at, seen = np.random.default_rng(0), (ctypes.c_int * 4)(), set()
    for case in range(600):
        tall, shorts = int(rng.integers(0, 900 if case < 400 else 4100)), int(rng.integers(0, 200)) if case % 2 else 0
        rounds = int(rng.integers(0, tall // 256 + 1)) if case >= 400 else 0
        blocks = rules.grid(tall + shorts + (0 if case % 4 < 2 else int(rng.integers(0, 3000))))
        covered = {}
        for b in range(blocks + 64):
            if not rules.part(b, blocks, tall, shorts, rounds, at):
                continue
            assert b < blocks and not (at[3] and at[2] >= 0)
            rows, cols = ([v] if v >= 0 else [0, 1] for v in (at[1], at[2]))
            seen.add((at[1] >= 0, at[2] >= 0, rounds > 0))
            for q in ((r, c) for r in rows for c in cols):
                covered[at[0], q] = covered.get((at[0], q), 0) + 1
        assert set(covered.values()) <= {1} and len(covered) == 4 * (tall + shorts)
    assert seen == {(*parts, dealt) for parts in ((False, False), (False, True), (True, True)) for dealt in (False, True)}


def test_launches_that_cut(rules):
    """Where part of a round is left over, by the rows that are expected; not in launches of whole rounds, nor of many."""
    for E, C, rows, up_to, NT in ((8, 5120, 4096, 1, 8), (8, 1100, 1100, 0, 8), (8, 2200, 2100, 1, 8), (32, 980, 784, 1, 3)):
        assert rules.cuts(E, C, rows, up_to, NT), (E, C, rows)
    for E, C, rows, up_to, NT in ((8, 4096, 4096, 0, 8), (64, 283, 283, 1, 2), (64, 2048, 2048, 1, 16), (128, 16384, 8192, 1, 16), (8, 1600, 1500, 1, 8)):
        assert not rules.cuts(E, C, rows, up_to, NT), (E, C, rows)


def cut_ends_later(E, rows, NT, apart):
    """An XCD's tiles in turn on 32 units, by a heap of the times at which these are free, whole and with the last, partial round in parts."""
    heights = -(-rows // 256)
    tall = ([True] * (E // 8 * NT * (heights - 1)) + [False] * (E // 8 * NT) if apart else
            [kind for _ in range(E // 8) for c in range(0, NT, 8) for kind, n in ((True, heights - 1), (False, 1)) for _ in range(n * min(8, NT - c))])
    over = len(tall) % 32
    def end(tasks):
        units = [0] * 32
        for t in tasks:
            heapq.heapreplace(units, units[0] + t)
        return max(units)
    first, rest = [20 if t else 8 for t in tall[:len(tall) - over]], tall[len(tall) - over:]
    if over > 8:
        parts = [13 if t else 11 for t in rest for _ in range(2)]
    else:
        parts = [10 if t else 6 for t in rest for _ in range(2)] + [10 for t in rest if t for _ in range(2)]
    return 20 * end(first + parts) >= 21 * end(first + [20 if t else 8 for t in rest])


def test_whole_tiles_where_short_ones_make_room(rules):
    """Every expert full, its last row tile of a few rows: products that took up to 1.17 times as long cut as whole stay whole, those that cutting makes faster
    are cut; everywhere as a plain walk over the tiles has it."""
    for E, rows, NT in ((16, 516, 8), (24, 516, 5), (8, 516, 15), (8, 528, 16), (8, 1028, 16), (16, 1027, 8), (8, 1537, 16)):
        assert not rules.cuts(E, rows, rows, 0, NT), (E, rows, NT)
    for E, rows, NT in ((32, 544, 4), (16, 272, 10), (24, 800, 3), (40, 784, 2), (32, 528, 3), (8, 612, 16), (8, 1152, 8), (12, 516, 8)):
        assert rules.cuts(E, rows, rows, 0, NT), (E, rows, NT)
    seen = set()
    for E, heights, NT in itertools.product((8, 16, 24, 40, 64), range(2, 14), range(1, 19)):
        n, tall = E * heights * NT // 8, E * (heights - 1) * NT
        if not 1 <= n % 32 <= 16 or n > 512 or (8 * n >= 1024 and heights >= 4):      # those deal whole groups, cut as they are
            continue
        apart = E * heights * NT <= 768 and 3 * E * NT <= tall <= 512 and -(-tall // 256) < -(-E * heights * NT // 256)
        for rows in (256 * heights - 255, 256 * heights - 224):
            assert rules.cuts(E, rows, rows, 0, NT) != cut_ends_later(E, rows, NT, apart), (E, rows, NT)
        seen.add((apart, n % 32 > 8, rules.cuts(E, rows, rows, 0, NT)))
    assert len(seen) >= 7


FILLS = {                                              # row tiles x 6 column tiles over 8 XCDs: tiles of an XCD
    "quarters": [2100, 2049, 2099, 2082, 2048 + 16],                    # 33 or 34: 1 or 2 beyond a whole round, of 1 to 52 rows
    "quarters alone": [256, 512, 129, 0, 257],                          # 4 or 5
    "halves": [1300, 1281, 1, 127, 700],                                # 12 or 13
    "halves of whole row tiles": [2048, 1536, 0, 0, 256],               # 11 or 12
    "uncut": [2100, 2100, 1400, 0, 64],                                 # 18 or 19
    "one row tile": [0, 0, 0, 0, 3],
}


def check_cut_products(rules, fills, act, M, H, bias=True):
    """All experts in one launch whose last round is cut against a launch for every expert on slabs of just its rows, none of which is cut: the sums run in the same order,
    so the bits are equal.  Slots past the fill are not written."""
    from paper_2206_03382_amd import moe
    E, C = 5, 2100
    assert rules.cuts(E, C, C, 1, H // 256)
    gen = torch.Generator(device="cuda").manual_seed(len(fills) + act)
    rand = lambda *shape, std=1.0: (torch.randn(shape, generator=gen, device="cuda") * std).to(torch.bfloat16)
    W1, W2, b1, b2 = rand(E, M, H, std=M ** -0.5), rand(E, H, M, std=H ** -0.5), rand(E, H), rand(E, M)
    if not bias:
        b1 = b2 = None
    T = 4000
    x, dY = rand(T, M), rand(E, C, M)
    slots = torch.randint(0, T, (E, C), generator=gen, device="cuda", dtype=torch.int32)
    c = torch.tensor(FILLS[fills], dtype=torch.int32, device="cuda")
    live = torch.arange(C, device="cuda")[None, :] < c[:, None]
    Z = torch.where(live[..., None], x[slots.long()], float("nan"))
    dY = torch.where(live[..., None], dY, float("nan"))
    hidden = torch.full((E, C, H), float("nan"), device="cuda", dtype=torch.bfloat16)
    Y = moe.expert_ffn(Z, W1, b1, W2, b2, act, counts=c, hidden=hidden)
    assert bool(hidden[~live].isnan().all())
    Yg = moe.expert_ffn_gather(x, slots, W1, b1, W2, b2, act, counts=c)
    Yt, hidden_t, pre = moe.expert_ffn_train(Z, W1, b1, W2, b2, act, counts=c)
    g = moe.expert_ffn_backward(Z, W1, b1, W2, hidden_t, dY, act, counts=c, pre=pre)
    for e, n in enumerate(FILLS[fills]):
        if n == 0:
            continue
        one = lambda t: t[e:e + 1, :n].contiguous()
        w = [None if t is None else t[e:e + 1] for t in (W1, b1, W2, b2)]
        want_Y, want_hidden, want_pre = moe.expert_ffn_train(one(Z), *w, act)
        want = moe.expert_ffn_backward(one(Z), w[0], w[1], w[2], want_hidden, one(dY), act, pre=want_pre)
        for name, got, ref in (("hidden", hidden, want_hidden), ("Y", Y, want_Y), ("gathered", Yg, want_Y), ("Yt", Yt, want_Y), ("hidden_t", hidden_t, want_hidden),
                               ("pre", pre, want_pre), ("dZ", g["dZ"], want["dZ"])):
            assert torch.equal(got[e, :n], ref[0]), (name, e, n)
        for name in ("dW1", "dW2"):                    # of dP and hidden: dP is a product with B transposed
            assert torch.equal(g[name][e], want[name][0]), (name, e, n)


def large_uncut(ffn_rules, rules, E, C, M, H):
    """Which of the products on C rows (forward, keeping its pre-activations, B transposed; over M) run on the large tile; those that a launch of one expert cuts."""
    tiles = (ffn_rules.tile(0, E, C, M, H, 0, 0), ffn_rules.tile_keeping_pre(E, C, M, H, 0, 0), ffn_rules.tile(1, E, C, M, H, 0, 0))
    return [t == 0 for t in tiles], [t == 0 and E == 1 and bool(rules.cuts(1, C, C, 0, H // 256)) for t in tiles]


@pytest.mark.gpu
@pytest.mark.parametrize("act", [O.ACT_RELU, O.ACT_GELU, O.ACT_SILU])
@pytest.mark.parametrize("fills", FILLS, ids=str)
def test_cut_products_have_the_same_bits(rules, ffn_rules, fills, act):
    """The forward (plain, gathered, keeping its pre-activations) and the products with B transposed."""
    assert large_uncut(ffn_rules, rules, 5, 2100, 1536, 1536)[0] == [True] * 3
    check_cut_products(rules, fills, act, 1536, 1536)


@pytest.mark.gpu
@pytest.mark.parametrize("fills", ["quarters", "halves", "one row tile"])
@pytest.mark.parametrize("K", [64, 128, 192, 256, 320])
def test_cut_products_of_short_reductions(rules, ffn_rules, K, fills):
    """One to five K-steps, fewer than, as many as and more than the rings of the parts hold (five and three): the product that keeps its pre-activations and the one with B transposed;
    without biases, too.  (Off the grid of 256 the derivative of GELU has two forms, by the tile, which differ in the last bit: ReLU there.)"""
    assert large_uncut(ffn_rules, rules, 5, 2100, K, 1536)[0][1:] == [True] * 2
    check_cut_products(rules, fills, O.ACT_GELU if K == 256 else O.ACT_RELU, K, 1536, bias=K != 192)


def test_single_launches_are_not_cut(rules, ffn_rules):
    """What the tests above compare with: a launch of one expert on any of their fills takes another tile, or leaves whole rounds."""
    for M in (64, 128, 192, 256, 320, 1536):
        for n in {n for f in FILLS.values() for n in f if n}:
            assert large_uncut(ffn_rules, rules, 1, n, M, 1536)[1] == [False] * 3, (M, n)
