"""Steps whose router sums what the tasks of the output projection leave: one task, a few more than the 32 that are loaded
together, the most there can be; one expert, counts that leave lanes without one, all 64.  Up to 64 tokens the expert kernels sort the
routed pairs themselves: token counts at the edges of a wave's share of pairs and of the token tiles; beyond, the histograms of
eight tokens (float32; 32 in bfloat16, whose router contracts there) feed the permutation: counts that end inside a histogram, a permutation
group and a token tile."""
import numpy as np
import pytest

import dinfer_inputs as di
import oracle
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, make_case

pytestmark = pytest.mark.gpu


# the last two: expert GEMMs and down projection of whole tasks (more tasks than compute units) and in pieces
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hidden,experts,top_k,width", [(64, 1, 1, 64), (2112, 33, 8, 64), (4096, 64, 5, 64), (128, 63, 7, 320), (320, 64, 8, 64)])
@pytest.mark.parametrize("n_seq,block", [(1, 1), (1, 9), (1, 32), (3, 11), (1, 63), (4, 16)])
def test_step_with_router_shares(n_seq, block, hidden, experts, top_k, width, dtype):
    check(n_seq, block, hidden, 1, experts, top_k, width, dtype)


# (float32: one head of 64 has a dense form of the output projection, which leaves shares; bfloat16: none does)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("hidden,n_heads,experts,top_k", [(64, 2, 1, 1), (2112, 2, 33, 8), (4096, 2, 64, 5), (320, 1, 64, 8)])
@pytest.mark.parametrize("n_seq,block", [(5, 13), (4, 24), (3, 43), (16, 33)])
def test_step_of_many_tokens_with_router_shares(n_seq, block, hidden, n_heads, experts, top_k, dtype):
    check(n_seq, block, hidden, n_heads, experts, top_k, 64, dtype)


def check(n_seq, block, hidden, n_heads, experts, top_k, width, dtype):
    # The float32 bar of the confidences (2e-5) is for logits as large as the float32 model's, 8 * 0.02 * sqrt(256): a logit's rounding error
    # grows with its size (about sqrt(hidden) * 6e-8 of it: 8e-5 for logits of 20) and moves a confidence c by up to c * (1 - c) times
    # twice that.  Wider models take a smaller scale, so that their logits are no larger; likewise in bfloat16, whose bars are those of
    # a hidden size of 2048 at scale 1.
    scale = 8.0 * min(1.0, (256 / hidden) ** 0.5) if dtype == "f32" else min(1.0, (2048 / hidden) ** 0.5)
    cfg = di.configs.scaled(di.model_preset("tiny"), hidden=hidden, n_heads=n_heads, head_dim=64, n_experts=experts, top_k=top_k, moe_inter=width,
                            vocab=300, dtype=dtype, logit_scale=scale)
    wl = di.Workload("shares", cfg, n_seq, block, 2, 30, threshold=0.9, seed_index=140 + n_seq)
    cfg, w, inp = make_case(wl)
    cap = int(inp.prefix_len.max()) + 2 * block + 16
    ora = OracleRun(cfg, w, inp, cap)
    gpu = GpuRun(cfg, w, inp, n_seq * block, cap)
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    got = gpu.step(wl.threshold)
    T = n_seq * block
    logits = gpu.logits(T).reshape(n_seq, block, cfg.vocab)
    routing = gpu.routing().reshape(cfg.n_layers, n_seq, block, cfg.top_k)
    tables = [gpu.ctx.debug_get(f, (n,), gpu.torch.int32).cpu().numpy() for f, n in ((3, experts), (4, experts + 1), (5, T * top_k))]
    for table, want in zip(tables, oracle.permutation(routing[-1].reshape(-1), experts)):
        assert np.array_equal(table, want)
    for s in range(n_seq):
        ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), int(inp.prefix_len[s]), wl.threshold, 0, routing[:, s], bars)
        compare_logits(ref["logits"], logits[s], bars)
        compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                     inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"], logits[s])
    gpu.close()
