"""Steps with several items of 128 rows per expert, whose expert GEMMs run in the form that shares an expert's weights on a die
(csrc/expert_plan.hpp), against the oracle: several task groups per item, light items beyond a round of the chip handed out in
pieces, experts of very different weight, one launch in that form and the other in plain order."""
import numpy as np
import pytest

import dinfer_inputs as di
import host_shim
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, make_case

pytestmark = pytest.mark.gpu

SHIM = """
#include "expert_plan.hpp"
using namespace dinfer;
extern "C" int tiles(int E, int n_pairs) { return expert_group_tiles(E, n_pairs); }
extern "C" int shared_form(int bf16, int E, int n_pairs, int groups) { return expert_shared(bf16 != 0, E, n_pairs, groups); }
extern "C" int pieces(int items, int light, int E, int n_pairs, int H, int I) {
  return expert_piece_items(items, light, expert_round_items(E, n_pairs, H, I));
}
"""


# (sequences, block length, experts, experts per token, expert width, items in pieces).  With as many experts per token as there
# are, every expert has every row: two full items and one of one or two tiles each, in rounds of 21 items.
SIZES = [(6, 44, 8, 8, 3008, 3), (15, 20, 8, 8, 3008, 3),
         (13, 43, 16, 8, 1600, None),       # up to five items per expert, some with a few rows or none
         (22, 48, 4, 1, 8192, None)]        # 32 task groups: gate/up in plain order in bf16, down shared


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_seq,block,experts,top_k,width,pieces", SIZES)
def test_step_with_shared_items(n_seq, block, experts, top_k, width, pieces, dtype, tmp_path):
    plan = host_shim.load(tmp_path, SHIM)
    tiny = di.model_preset("tiny")
    cfg = di.configs.scaled(tiny, n_heads=2, head_dim=128, n_experts=experts, top_k=top_k, moe_inter=width, vocab=700, dtype=dtype,
                            logit_scale=8.0 if dtype == "f32" else 1.0)
    wl = di.Workload("shared", cfg, n_seq, block, 3, 70, precommit=True, threshold=0.9, seed_index=130 + n_seq)
    cfg, w, inp = make_case(wl)
    cap = int(inp.prefix_len.max()) + 2 * block + 16
    ora = OracleRun(cfg, w, inp, cap)
    gpu = GpuRun(cfg, w, inp, n_seq * block, cap)
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    got = gpu.step(wl.threshold)
    logits = gpu.logits(n_seq * block).reshape(n_seq, block, cfg.vocab)
    routing = gpu.routing()
    # the case is what it says: the form, and the light items that every layer hands out in pieces
    n_pairs, groups = n_seq * block * top_k, [(width // 32 + 7) // 8, (cfg.hidden // 64 + 7) // 8]
    bf = int(dtype == "bf16")
    assert plan.tiles(experts, n_pairs) == 4 and plan.shared_form(bf, experts, n_pairs, groups[1])
    assert plan.shared_form(bf, experts, n_pairs, groups[0]) == (0 if bf and groups[0] == 32 else 1)
    for l in range(cfg.n_layers):
        rows = np.bincount(routing[l].reshape(-1), minlength=experts)
        items, light = int((rows // 128 + (rows % 128 > 0)).sum()), int(((rows % 128 > 0) & (rows % 128 <= 64)).sum())
        assert pieces is None or plan.pieces(items, light, experts, n_pairs, cfg.hidden, width) == pieces
    routing = routing.reshape(cfg.n_layers, n_seq, block, cfg.top_k)
    for s in range(n_seq):
        ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), int(inp.prefix_len[s]), wl.threshold, 0,
                                    routing[:, s], bars)
        compare_logits(ref["logits"], logits[s], bars)
        compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                     inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"], logits[s])
    gpu.close()
