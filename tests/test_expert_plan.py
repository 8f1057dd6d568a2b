"""How the routed rows of more than 64 tokens are dealt out (csrc/expert_plan.hpp), compiled for the host: whatever the
routing, the grid of the expert GEMMs holds every whole item and every piece, and no more pieces than a routing can give."""
import ctypes

import numpy as np
import pytest

import host_shim

SHIM = """
#include "expert_plan.hpp"
using namespace dinfer;
extern "C" void plan(int E, int n_pairs, int H, int I, int* o) {
  o[0] = expert_group_tiles(E, n_pairs), o[1] = expert_round_items(E, n_pairs, H, I);
  o[2] = expert_work_items(E, n_pairs, o[0]), o[3] = expert_most_piece_items(E, n_pairs, H, I);
}
extern "C" int unit_wgs(int n, int groups) { return expert_unit_wgs(n, groups); }
extern "C" void units(int n_wgs, int heavy, int full, int n, int groups, int* o) {
  for (int i = 0; i < n_wgs; ++i) {
    const ExpertUnit u = expert_unit(i, heavy, full, n, groups);
    o[2 * i] = u.item, o[2 * i + 1] = u.group;
  }
}
extern "C" int shared_form(int bf16, int E, int n_pairs, int groups) { return expert_shared(bf16 != 0, E, n_pairs, groups); }
extern "C" int piece_items(int items, int light, int round) { return expert_piece_items(items, light, round); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_shim.load(tmp_path_factory.mktemp("expert_plan"), SHIM)


def _plan(lib, E, n_pairs, H, I):
    o = (ctypes.c_int * 4)()
    lib.plan(E, n_pairs, H, I, o)
    return list(o)


def _items(counts, rows_per):
    """Items of a routing and the light ones (up to two tiles of 32 rows), as the permutation kernel lists them."""
    full, rem = counts // rows_per, counts % rows_per
    light = int(((rem > 0) & (rem <= 64)).sum()) + (int(full.sum()) if rows_per <= 64 else 0)
    return int(full.sum() + (rem > 0).sum()), light


@pytest.mark.parametrize("E,k,H,I", [(64, 8, 2048, 1024), (64, 8, 64, 64), (48, 1, 128, 192), (16, 2, 2048, 4096),
                                     (8, 2, 256, 512), (40, 8, 1024, 2048), (1, 1, 4096, 64), (5, 3, 4096, 8192)])
def test_grid_holds_every_routing(lib, E, k, H, I):
    rng = np.random.default_rng(E * 1000 + k)
    for T in [65, 66, 96, 97, 128, 192, 193, 200, 256, 384, 500, 512, 777, 1024, 1298, 2048, 4096]:
        n_pairs = T * k
        tiles, rnd, most_items, most_pieces = _plan(lib, E, n_pairs, H, I)
        assert rnd >= 1 and 0 <= most_pieces <= rnd
        for trial in range(60):
            conc = [0.05, 0.3, 1.0, 10.0, 1000.0][trial % 5]
            if trial == 0:      # as many experts as possible one row beyond a whole number of groups
                counts = np.zeros(E, dtype=np.int64)
                left = n_pairs
                for e in range(E):
                    take = min(left, T, tiles * 32 * ((n_pairs // E) // (tiles * 32)) + 1)
                    counts[e] = take
                    left -= take
                for e in range(E):
                    add = min(left, T - counts[e])
                    counts[e] += add
                    left -= add
            else:
                counts = np.minimum(rng.multinomial(n_pairs, rng.dirichlet(np.full(E, conc))), T)
            assert counts.max() <= T
            items, light = _items(counts, tiles * 32)
            pieces = lib.piece_items(items, light, rnd)
            assert items <= most_items and 0 <= pieces <= min(most_pieces, light, items)
            assert pieces == 0 or items > rnd


def test_pieces_are_few(lib):
    assert lib.piece_items(64, 64, 64) == 0                       # exactly one round
    assert lib.piece_items(64 + 24, 64, 64) == 24                 # three eighths of another
    assert lib.piece_items(64 + 25, 64, 64) == 0
    assert lib.piece_items(2 * 64 + 5, 64, 64) == 5
    assert lib.piece_items(64 + 9, 8, 64) == 0                    # one of them has more than two tiles
    # a forward whose routing cannot exceed a round asks for no workgroups of pieces
    assert _plan(lib, 48, 1298, 128, 192)[3] == 0
    assert _plan(lib, 64, 8 * 256, 2048, 1024)[3] == 64 + 2048 // 128 - 64


@pytest.mark.parametrize("groups", [1, 2, 3, 4, 11, 22, 31, 43])
def test_shared_items_go_to_the_dies_in_equal_runs(lib, groups):
    """Workgroup i runs on die i % 8.  Every (item, task group) pair is taken once; of the items of each weight, and of all, no
    die has more than one pair more than another, so that none runs a round of workgroups longer; a die takes the heavy
    ones first and has a run of consecutive pairs of each kind, so that the task groups of an item meet on it."""
    rng = np.random.default_rng(groups)
    for trial in range(200):
        n = [1, 2, 7, 8, 9, 23, 24, 48, 331][trial] if trial < 9 else int(rng.integers(1, 400))
        heavy = int(rng.integers(0, n + 10))     # the list may go on behind the n items (with the ones handed out in pieces)
        full = heavy + int(rng.integers(0, n + 10))
        n_wgs = lib.unit_wgs(n, groups)
        assert n_wgs <= (n + 7) * groups         # the rows that the launch adds to the grid
        o = (ctypes.c_int * (2 * n_wgs))()
        lib.units(n_wgs, heavy, full, n, groups, o)
        u = np.array(o).reshape(-1, 2)
        pair = np.where(u[:, 0] >= 0, u[:, 0] * groups + u[:, 1], -1)
        assert np.array_equal(np.sort(pair[pair >= 0]), np.arange(n * groups))
        assert np.all((u[:, 1] >= 0) & (u[:, 1] < groups))
        kind = (u[:, 0] >= heavy).astype(int) + (u[:, 0] >= full)
        dies = [[(kind[i], pair[i]) for i in range(d, n_wgs, 8) if pair[i] >= 0] for d in range(8)]
        assert max(map(len, dies)) - min(map(len, dies)) <= 1
        for k in range(3):
            runs = [[p for kk, p in die if kk == k] for die in dies]
            assert max(map(len, runs)) - min(map(len, runs)) <= 1
            assert all(r == list(range(r[0], r[0] + len(r))) for r in runs if r)
        assert all([k for k, _ in die] == sorted(k for k, _ in die) for die in dies)


def test_shared_form_where_items_meet_on_a_die(lib):
    assert lib.shared_form(1, 64, 64 * 256, 4) and not lib.shared_form(1, 64, 64 * 256 - 1, 4)
    assert lib.shared_form(1, 8, 8 * 300, 31) and not lib.shared_form(1, 8, 8 * 300, 32)    # 32 groups fill a die ...
    assert lib.shared_form(1, 8, 8 * 300, 33) and not lib.shared_form(1, 8, 8 * 300, 40)
    assert lib.shared_form(0, 8, 8 * 300, 32) and not lib.shared_form(0, 8, 8 * 255, 4)      # ... in bf16
