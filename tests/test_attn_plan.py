"""Which form of attention a forward takes (csrc/attn_plan.hpp), compiled for the host."""
import ctypes

import pytest

import host_shim

SHIM = """
#include "attn_plan.hpp"
extern "C" int groups(const int* off, int n_seq, int n_heads, int from_zero) {
  return dinfer::attn_rows_groups(off, n_seq, n_heads, from_zero != 0);
}
"""


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    lib = host_shim.load(tmp_path_factory.mktemp("attn_plan"), SHIM)

    def of(lens, n_heads, from_zero):
        off = [0]
        for n in lens:
            off.append(off[-1] + n)
        return lib.groups((ctypes.c_int * len(off))(*off), len(lens), n_heads, int(from_zero))
    return of


def test_prompts_that_fill_the_chip_take_the_rows_form(groups):
    assert groups([2048], 16, True) == 16
    assert groups([1024], 16, True) == 0                  # 128 workgroups
    assert groups([1811, 333, 825, 1318], 16, True) == 15 + 3 + 7 + 11
    assert groups([385, 416, 447, 97], 32, True) == 4 + 4 + 4 + 1
    assert groups([64] * 32, 16, True) == 0               # two of four waves without queries
    assert groups([96] * 16, 16, True) == 16


def test_runs_behind_cached_prefixes_keep_the_splitting_form(groups):
    for run in (65, 80, 96, 128):                         # vicinity steps: blocks of 64 with up to 64 neighbours
        for n_seq in (8, 16, 64):
            assert groups([run] * n_seq, 16, False) == 0
