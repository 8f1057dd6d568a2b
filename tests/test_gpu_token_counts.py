"""Steps at the token counts where the expert GEMMs and the LM head change their form: the first count above the
64-token forms, both sides of the line between two and four row tiles per work item, token groups of unequal size."""
import numpy as np
import pytest

import dinfer_inputs as di
import oracle
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, make_case
from test_gpu_tiny import _skew_router

pytestmark = pytest.mark.gpu

# (sequences, block length, skewed router, experts, expert width).  64 experts, 8 per token: two-tile work items up to
# 192 tokens.  Expert width 2048: a round of the chip is 32 items, and the items beyond it (one or two tiles each) are
# handed out in pieces.
SIZES = [(5, 13, False, 64, 192), (3, 32, False, 64, 192), (4, 32, True, 64, 192), (5, 32, False, 64, 192),
         (5, 32, True, 64, 192), (3, 64, False, 64, 192), (4, 49, False, 64, 192), (4, 50, True, 64, 192),
         (4, 30, False, 40, 2048), (5, 13, False, 36, 2112), (4, 33, False, 40, 2048), (5, 40, False, 40, 2048), (9, 60, False, 35, 2112), (16, 64, False, 64, 2048)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_seq,block,skew,experts,width", SIZES)
def test_step_at_token_count(n_seq, block, skew, experts, width, dtype):
    tiny = di.model_preset("tiny")
    cfg = di.configs.scaled(tiny, n_heads=2, head_dim=128, n_experts=experts, top_k=8, moe_inter=width, vocab=1100, dtype=dtype,
                            logit_scale=8.0 if dtype == "f32" else 1.0)
    wl = di.Workload("tokens", cfg, n_seq, block, 3, 70, precommit=True, threshold=0.9, seed_index=50 + n_seq)
    cfg, w, inp = make_case(wl)
    if skew:
        _skew_router(cfg, w)
    cap = int(inp.prefix_len.max()) + 2 * block + 16
    ora = OracleRun(cfg, w, inp, cap)
    gpu = GpuRun(cfg, w, inp, n_seq * block, cap)
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    got = gpu.step(wl.threshold)
    logits = gpu.logits(n_seq * block).reshape(n_seq, block, cfg.vocab)
    routing = gpu.routing().reshape(cfg.n_layers, n_seq, block, cfg.top_k)
    # the token -> expert permutation of the last layer is a stable counting sort of its routing
    n_pairs = n_seq * block * cfg.top_k
    tables = [gpu.ctx.debug_get(w, (n,), gpu.torch.int32).cpu().numpy() for w, n in ((3, experts), (4, experts + 1), (5, n_pairs))]
    for got_table, want in zip(tables, oracle.permutation(routing[-1].reshape(-1), cfg.n_experts)):
        assert np.array_equal(got_table, want)
    for s in range(n_seq):
        ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), int(inp.prefix_len[s]), wl.threshold, 0,
                                    routing[:, s], bars)
        compare_logits(ref["logits"], logits[s], bars)
        compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                     inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"], logits[s])
    gpu.close()
