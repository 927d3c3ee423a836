import ctypes
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)


def pytest_configure(config):
    config.addinivalue_line("markers", "gpu: needs a real MI355X (run with -m gpu)")


@pytest.fixture(scope="session")
def golden_dir():
    return os.path.join(ROOT, "tests", "golden")


RULES_SOURCE = r"""
#include "paper_2206_03382_amd/csrc/ffn_rules.h"
#include "paper_2206_03382_amd/csrc/gate_rules.h"
extern "C" {
int64_t grid(int64_t E, int64_t C, int64_t tile, int64_t NT, int64_t total, int shorts_last) {
  return moe::tile_grid(NT, moe::live_row_tiles(E, C, total, tile), shorts_last);
}
int equal_tile(int b, int E, int MT, int NT, int* at) {
  moe::TileAt t;
  if (!moe::equal_tile(b, E, MT, NT, t)) return 0;
  at[0] = t.e; at[1] = t.mt; at[2] = t.nt;
  return 1;
}
// find_tile, one expert behind the other instead of 64 lanes at a time
int tile_at(int b, int E, const int* rows, int tile_rows, int NT, int shift, int shorts_last, int* at) {
  const int gs = moe::kGroupShift + shift;
  int all_rows = 0, all_tiles = 0, without = 0, tall = 0, shorts = 0, full = 0, upto = 0, groups = 0, short_upto = 0;
  for (int e = 0; e < E; ++e) {
    all_rows += rows[e];
    all_tiles += moe::tall_row_tiles(rows[e], tile_rows, false) * NT;
    without += moe::tall_row_tiles(rows[e], tile_rows, true) * NT;
  }
  bool apart = moe::may_open_a_round(all_tiles, shift) && moe::opens_a_round(without, all_tiles, shift);
  for (int e = 0; e < E; ++e) apart = apart || moe::far_above_mean(rows[e], E, all_rows);
  apart = apart && shorts_last;
  for (int e = 0; e < E; ++e) {
    const int mt = moe::tall_row_tiles(rows[e], tile_rows, apart);
    tall += mt * NT;
    full += mt * NT >> gs;
    shorts += rows[e] > mt * tile_rows ? NT : 0;
  }
  const int rounds = moe::deals_groups(tall, E, NT, shift) ? full >> 3 : 0;
  const moe::TileSpot s = moe::tile_spot(b, tall, shorts, rounds, gs);
  if (s.part == moe::kNoTile) return 0;
  for (int e = 0; e < E; ++e) {
    const int mt = moe::tall_row_tiles(rows[e], tile_rows, apart), all = mt * NT;
    upto += all;
    groups += all >> gs;
    short_upto += rows[e] > mt * tile_rows ? NT : 0;
    const int inc = s.part == moe::kShortTile ? short_upto : (s.part == moe::kDealtTile ? groups : upto - ((groups < rounds * 8 ? groups : rounds * 8) << gs));
    if (inc <= s.at) continue;
    const int back = s.at - inc;
    moe::TileAt t = {e, mt, NT + back};
    if (s.part != moe::kShortTile) t = moe::tile_in_expert(e, s.part == moe::kDealtTile ? ((back + (all >> gs)) << gs) + (b / 8 & ((1 << gs) - 1)) : all + back, mt, NT);
    at[0] = t.e; at[1] = t.mt; at[2] = t.nt;
    return 1 + s.part;
  }
  return -1;
}
int half_shift() { return moe::kHalfGroupShift; }
int tile(int mode, int64_t E, int64_t C, int64_t K, int64_t N, int64_t rows_hint, int64_t gather_rows) {
  return (int)moe::tile_of(mode, E, C, K, N, rows_hint, gather_rows, false);
}
int tile_keeping_pre(int64_t E, int64_t C, int64_t K, int64_t N, int64_t rows_hint, int64_t gather_rows) {
  return (int)moe::tile_of(moe::kNN, E, C, K, N, rows_hint, gather_rows, true);
}
double tile_cost(int tile, int mode, int64_t E, int64_t C, int64_t K, int64_t N, int64_t rows_hint, int64_t gather_rows) {
  return moe::tile_cost((moe::Tile)tile, mode, E, C, moe::mean_or(rows_hint, mode == moe::kTN ? K : C), K, N, gather_rows > 0);
}
int cuts(int64_t E, int64_t C, double rows, int up_to, int64_t NT) { return moe::cuts_last_round(E, C, rows, up_to, NT); }
int colsum_streams(int64_t E, double rows, int64_t b1, int64_t b2) { return moe::colsum_streams(E, rows, b1, b2); }
int split(int64_t E, int64_t C, int64_t K, int64_t N) { return moe::fp32_split(E, C, K, N); }
int dx_tokens(int64_t T, int64_t row_bytes) { return moe::gate_dx_tokens(T, row_bytes); }
int64_t backward_tokens(int64_t T, int64_t E, int bias) { return moe::gate_backward_token_block(T, E, bias); }
int64_t wide_logits(int64_t T, int64_t E, int vecw) { return moe::gate_logits_wide_experts(T, E, vecw); }
int one_block(int64_t T, int64_t E, int k, int64_t marked_C) { return moe::gate_in_one_block(T, E, k, marked_C); }
int64_t lane_topk_blocks(int64_t E, int k, int64_t M) { return moe::gate_lane_topk_blocks(E, k, M); }
int one_launch(int64_t T, int64_t E, int k) { return moe::slots_in_one_launch((T + 63) / 64, E, k); }
}
"""


@pytest.fixture(scope="session")
def ffn_rules(tmp_path_factory):
    """The host rules of the grouped GEMM: grid(), equal_tile(), tile_at(), tile(), whose results are numbered as the enum in csrc/ffn_rules.h is, the same for a
    product that keeps its pre-activations, tile_cost(), cuts(), colsum_streams() and split(); and of the gate: one_block(), lane_topk_blocks(), one_launch(), dx_tokens(), backward_tokens(), wide_logits()."""
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text(RULES_SOURCE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", ROOT, str(d / "rules.cpp"), "-o", str(d / "rules.so")], check=True)
    lib = ctypes.CDLL(str(d / "rules.so"))
    lib.grid.restype, lib.grid.argtypes = ctypes.c_int64, [ctypes.c_int64] * 5 + [ctypes.c_int]
    lib.equal_tile.restype, lib.equal_tile.argtypes = ctypes.c_int, [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int)]
    lib.tile_at.restype = ctypes.c_int
    lib.tile_at.argtypes = [ctypes.c_int] * 2 + [ctypes.POINTER(ctypes.c_int)] + [ctypes.c_int] * 4 + [ctypes.POINTER(ctypes.c_int)]
    lib.tile.restype, lib.tile.argtypes = ctypes.c_int, [ctypes.c_int] + [ctypes.c_int64] * 6
    lib.cuts.restype, lib.cuts.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_double, ctypes.c_int, ctypes.c_int64]
    lib.colsum_streams.restype, lib.colsum_streams.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_double] + [ctypes.c_int64] * 2
    lib.split.restype, lib.split.argtypes = ctypes.c_int, [ctypes.c_int64] * 4
    lib.tile_keeping_pre.restype, lib.tile_keeping_pre.argtypes = ctypes.c_int, [ctypes.c_int64] * 6
    lib.tile_cost.restype, lib.tile_cost.argtypes = ctypes.c_double, [ctypes.c_int] * 2 + [ctypes.c_int64] * 6
    lib.one_block.restype, lib.one_block.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int64]
    lib.lane_topk_blocks.restype, lib.lane_topk_blocks.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int, ctypes.c_int64]
    lib.one_launch.restype, lib.one_launch.argtypes = ctypes.c_int, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    lib.dx_tokens.restype, lib.dx_tokens.argtypes = ctypes.c_int, [ctypes.c_int64] * 2
    lib.backward_tokens.restype, lib.backward_tokens.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    lib.wide_logits.restype, lib.wide_logits.argtypes = ctypes.c_int64, [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return lib


@pytest.fixture
def progress(capsys):
    """print() that pytest does not capture, so that a long test shows its steps while it runs."""
    def say(msg):
        with capsys.disabled():
            print(f"\n[progress] {msg}", end="", flush=True)
    return say
