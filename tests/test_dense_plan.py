"""Which form the dense projections of more than 64 tokens take (csrc/dense_plan.hpp), compiled for the host."""
import ctypes

import pytest

import host_shim

SHIM = """
#include "dense_plan.hpp"
extern "C" int form(int bf16, int n_tasks, int T) {
  const dinfer::DenseForm f = dinfer::dense_form(bf16 != 0, n_tasks, T);
  return 10 * f.tasks + f.tiles;
}
extern "C" int groups(int bf16, int n_tasks, int T) { return dinfer::dense_form(bf16 != 0, n_tasks, T).groups; }
"""


@pytest.fixture(scope="module")
def form(tmp_path_factory):
    lib = host_shim.load(tmp_path_factory.mktemp("dense_plan"), SHIM)
    return lambda dtype, n_tasks, T: divmod(lib.form(int(dtype == "bf16"), n_tasks, T), 10)


def test_two_tiles_follow_the_type(form):
    assert form("bf16", 96, 320) == (4, 1) and form("bf16", 96, 352) == (4, 2)        # 240 and 264 workgroups of one tile
    assert form("f32", 48, 704) == (4, 1) and form("f32", 48, 768) == (4, 1)          # 264 and 288
    assert form("f32", 144, 256) == (4, 1) and form("f32", 96, 416) == (4, 2)         # 288; 312, 168 of two tiles
    assert form("f32", 48, 832) == (4, 1) and form("f32", 48, 896) == (4, 2)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_two_tasks_where_four_leave_the_chip_idle(form, dtype):
    assert form(dtype, 96, 96) == (2, 1) and form(dtype, 96, 160) == (2, 1) and form(dtype, 96, 192) == (4, 1)
    assert form(dtype, 32, 512) == (2, 1) and form(dtype, 32, 560) == (4, 1)


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    lib = host_shim.load(tmp_path_factory.mktemp("dense_groups"), SHIM)
    return lambda dtype, n_tasks, T: lib.groups(int(dtype == "bf16"), n_tasks, T)


def test_eight_tasks_from_the_second_round_of_four(form):
    assert form("bf16", 96, 640) == (4, 2) and form("bf16", 96, 641) == (8, 4)        # 24 x 10 and 24 x 11 workgroups
    assert form("bf16", 32, 2048) == (4, 2) and form("bf16", 32, 2049) == (8, 4)
    assert form("bf16", 36, 4000) == (8, 4) and form("bf16", 33, 4000) == (4, 2) and form("f32", 96, 4000) == (4, 2)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_token_groups_cover_every_tile(form, groups, dtype):
    """Of the form with four tiles, group g takes tiles tiles*g/n .. tiles*(g+1)/n: at least one and at most four."""
    for n_tasks in (1, 2, 6, 8, 16, 32, 33, 48, 64, 96, 144, 192):
        for T in list(range(65, 2200, 31)) + [4287, 8192, 30001]:
            tiles, n = (T + 31) // 32, groups(dtype, n_tasks, T)
            most = form(dtype, n_tasks, T)[1]
            if most < 4:
                assert n == (tiles + most - 1) // most, (n_tasks, T)
                continue
            size = {tiles * (g + 1) // n - tiles * g // n for g in range(n)}
            assert min(size) >= 1 and max(size) <= 4 and tiles * n < 2 ** 32, (n_tasks, T)


HALF_SHIM = """
#include "dense_plan.hpp"
extern "C" int half(int bf16, int K, int T, int n_tasks) { return dinfer::half_applies(bf16 != 0, K, T, n_tasks); }
extern "C" int slices(int bf16, int K, int T, int n_tasks) { return dinfer::ksplit_slices(bf16 != 0, K, T, n_tasks); }
"""


def test_half_tasks_replace_two_slices(tmp_path):
    """Every width, token and task count that takes half tasks would have taken two slices (the order of the sums), in whole
    shares of 8 or 16 k-steps for the eight waves; float32, more than 32 tokens, and fewer than 64 tasks do not."""
    lib = host_shim.load(tmp_path, HALF_SHIM)
    taken = set()
    for K in range(64, 4097, 64):
        for n_tasks in range(1, 260):
            for T in (1, 11, 32, 33, 64, 65):
                assert not lib.half(0, K, T, n_tasks)
                if lib.half(1, K, T, n_tasks):
                    assert lib.slices(1, K, T, n_tasks) == 2 and K // 16 in (8 * 8, 8 * 16) and T <= 32
                    taken.add((K, n_tasks))
    assert taken == {(K, n) for K in (1024, 2048) for n in range(64, 128)}
