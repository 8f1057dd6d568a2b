"""The LM head's division of the vocabulary (csrc/lm_plan.hpp), compiled for the host: at every vocabulary size the whole
groups and the pieces cover each task exactly once, and the number of partials the merge reads per row is the number of
workgroups (above 64 tokens: waves) that write one."""
import ctypes

import numpy as np
import pytest

import host_shim

SHIM = """
#include "lm_plan.hpp"
extern "C" void plans(int T, int v0, int n, int* out) {
  for (int i = 0; i < n; ++i) {
    const dinfer::LmPlan p = dinfer::lm_plan(v0 + i, T);
    int* o = out + 6 * i;
    o[0] = p.tasks, o[1] = p.ww, o[2] = p.whole, o[3] = p.first_piece, o[4] = p.parts, o[5] = dinfer::lm_head_most_parts(v0 + i);
  }
}
extern "C" int compact(int bf16, int T) { return dinfer::lm_compact(bf16 != 0, T); }
extern "C" int half(int bf16, int T) { return dinfer::lm_half(bf16 != 0, T); }
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    lib = host_shim.load(tmp_path_factory.mktemp("lm_plan"), SHIM)

    def table(T, v0, n):
        out = np.empty((n, 6), dtype=np.int32)
        lib.plans(T, v0, n, out.ctypes.data_as(ctypes.c_void_p))
        return out.T.astype(np.int64)
    return table


@pytest.mark.parametrize("T", [1, 32, 33, 48, 64, 65, 4096])
def test_every_vocabulary(plans, T):
    tasks, ww, whole, first, parts, most = plans(T, 2, 1 << 20)
    vocab = np.arange(2, 2 + (1 << 20))
    ok = tasks == -(-vocab // 64)
    ok &= (first == np.minimum(tasks, whole * ww)) & (whole >= 0)      # the whole groups take the tasks in front of first
    ok &= (whole == 0) | ((whole - 1) * ww < tasks)                    # none of them is empty
    pieces = tasks - first                                             # the others one workgroup each
    ok &= pieces >= 0
    ok &= parts == (whole + pieces if T <= 64 else whole * ww)
    ok &= (parts <= most) & (parts > 0)
    if T > 64:
        ok &= pieces == 0
    assert ok.all(), "vocabulary %d" % vocab[~ok][0]


def test_pieces_are_few(plans):
    """33 to 64 tokens: the groups of four tasks beyond a round of 512 go out task by task where they are at most a fifth of
    one, whole otherwise."""
    for rounds in (1, 2, 3):
        for over, in_pieces in ((0, 0), (1, 1), (102, 102), (103, 0), (187, 0), (255, 0), (511, 0)):
            tasks, ww, whole, first, parts, _ = plans(48, (512 * rounds + over) * 256, 1)[:, 0]
            assert ww == 4 and whole == 512 * rounds + over - in_pieces and tasks - first == 4 * in_pieces, (rounds, over)


def test_high_plane_of_many_bf16_tokens(tmp_path):
    lib = host_shim.load(tmp_path, SHIM)
    assert [lib.compact(1, T) for T in (1, 64, 65, 4096)] == [0, 0, 1, 1]
    assert [lib.compact(0, T) for T in (64, 65, 4096)] == [0, 0, 0]


def test_half_tasks_of_five_six_and_ten_token_tiles(tmp_path):
    lib = host_shim.load(tmp_path, SHIM)
    assert [T for T in range(1, 2000) if lib.half(1, T)] == list(range(129, 193)) + list(range(289, 321))
    assert not any(lib.half(0, T) for T in range(1, 2000))
