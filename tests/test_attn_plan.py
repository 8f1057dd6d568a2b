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


def test_prompts_of_one_length_a_little_beyond_a_round_keep_the_splitting_form(groups):
    assert groups([2048], 16, True) == 16 and groups([2049], 16, True) == 0            # 256 and 272 workgroups
    assert groups([2560], 16, True) == 0 and groups([2688], 16, True) == 21            # 320 and 336
    assert groups([1132], 32, True) == 9                                               # 288, but a short walk
    assert groups([1536, 1024, 512], 16, True) == 24 and groups([1408, 1280], 16, True) == 21
    assert groups([1152, 1152], 16, True) == 18 and groups([2304, 2304], 8, True) == 0
    assert groups([6016], 8, True) == 0 and groups([6252], 8, True) == 49              # 376 and 392 workgroups, a long walk
    assert groups([8300], 8, True) == 0 and groups([4332], 16, True) == 0 and groups([4716], 16, True) == 37
