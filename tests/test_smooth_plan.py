"""How the expected-embedding contraction is cut (csrc/smooth_plan.hpp), compiled for the host: the partial sums fit the room
they are given, and the launch fills the chip whatever the vocabulary, as long as it has chunks to deal out."""
import ctypes

import numpy as np
import pytest

import host_shim

SHIM = """
#include "smooth_plan.hpp"
extern "C" void plan(int H, int V, int ks, int T, int* o) {
  const dinfer::SmoothPlan p = dinfer::smooth_plan(H, V, ks, T);
  o[0] = p.wt, o[1] = p.task_groups, o[2] = p.token_groups, o[3] = p.pairs, o[4] = p.slices, o[5] = p.in_logits;
}
extern "C" int item(int i, int token_groups, int task_groups, int slices) {
  const dinfer::SmoothItem t = dinfer::smooth_item(i, token_groups, task_groups, slices);
  return t.valid ? (t.token_group * task_groups + t.task_group) * slices + t.slice : -1;
}
extern "C" long long part_bytes(int H, int V, int ks, int max_tokens) {
  return (long long)dinfer::smooth_part_bytes(H, V, ks, max_tokens);
}
"""
HIDDEN = [64, 128, 256, 320, 1024, 2048, 2880, 4096]
VOCAB = [2, 100, 1001, 4096, 5000, 32000, 50257, 157184, 262000]
TOKENS = [1, 11, 32, 33, 64, 65, 96, 128, 129, 160, 512, 1024, 1280, 4096]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    so = host_shim.load(tmp_path_factory.mktemp("smooth_plan"), SHIM)
    so.part_bytes.restype = ctypes.c_longlong
    return so


def _plan(lib, H, V, ks, T):
    o = (ctypes.c_int * 6)()
    lib.plan(H, V, ks, T, o)
    return dict(zip(("wt", "task_groups", "token_groups", "pairs", "slices", "in_logits"), o))


@pytest.mark.parametrize("ks", [16, 8])       # features of a k-step: bf16, float32
@pytest.mark.parametrize("H", HIDDEN)
def test_partial_sums_fit_and_the_chip_is_filled(lib, H, ks):
    for V in VOCAB:
        room = {m: lib.part_bytes(H, V, ks, m) for m in TOKENS}
        for T in TOKENS:
            p = _plan(lib, H, V, ks, T)
            assert p["wt"] in (1, 2, 4) and p["wt"] * p["token_groups"] * 32 >= T
            assert p["pairs"] == -(-V // (ks * 8))                      # nothing is contracted for padding
            assert 1 <= p["slices"] <= p["pairs"]                       # every slice has whole chunks for both teams
            if p["slices"] > 1:
                need = p["slices"] * T * H * 4
                for m in TOKENS:                                        # in any context that takes T tokens
                    assert m < T or need <= (T * V * 4 if p["in_logits"] else room[m]), (V, T, m)
            units = p["task_groups"] * p["token_groups"]
            assert p["slices"] * units <= max(256, units)
            # no compute unit idle for want of slices: rounding to eights and whole units costs less than half
            assert p["slices"] * units > min(128, units * (p["pairs"] // 2) // 2 - 1), (V, T, p)


def test_vocabulary_of_few_rows_of_features(lib):
    p = _plan(lib, 2048, 32000, 16, 32)
    assert p["slices"] * p["task_groups"] == 256 and not p["in_logits"]
    assert lib.part_bytes(2048, 32000, 16, 32) == 8 << 20
    assert lib.part_bytes(2048, 157184, 16, 512) == 0


@pytest.mark.parametrize("token_groups,task_groups,slices", [(1, 8, 32), (1, 3, 5), (1, 1, 1), (2, 8, 16), (3, 2, 7), (12, 10, 2),
                                                             (24, 10, 1), (32, 16, 1), (5, 1, 48)])
def test_items_over_the_dies(lib, token_groups, task_groups, slices):
    """Workgroup i runs on die i % 8: every item once, and as many on each die as on any other, or one fewer."""
    total = token_groups * task_groups * slices
    seen = [lib.item(i, token_groups, task_groups, slices) for i in range(-(-total // 8) * 8)]
    assert sorted(v for v in seen if v >= 0) == list(range(total))
    on_die = [sum(v >= 0 for v in seen[d::8]) for d in range(8)]
    assert max(on_die) == -(-total // 8)
