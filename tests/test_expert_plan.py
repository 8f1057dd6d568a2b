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
extern "C" int item_place(int i, int n, int stride) { return expert_item_place(i, n, stride); }
extern "C" int next_place(int p, int n, int stride) { return expert_next_place(p, n, stride); }
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


@pytest.mark.parametrize("stride", [1, 8])
def test_items_have_places_of_their_own(lib, stride):
    """Consecutive items lie a stride apart but where the list wraps, so that an expert's items run on one die."""
    for n in list(range(1, 40)) + [63, 64, 65, 331, 509]:
        places = [lib.item_place(i, n, stride) for i in range(n)]
        assert sorted(places) == list(range(n))
        assert places[1:] == [lib.next_place(p, n, stride) for p in places[:-1]]
        assert sum(b != a + stride for a, b in zip(places, places[1:])) < stride
