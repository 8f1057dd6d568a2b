"""Steps of up to 64 tokens, whose router sums what the tasks of the output projection leave and whose expert kernels sort the
routed pairs themselves: one task, a few more than the 32 that are loaded together, the most there can be; one expert, counts that
leave lanes without one, all 64; token counts at the edges of a wave's share of pairs and of the token tiles."""
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
    cfg = di.configs.scaled(di.model_preset("tiny"), hidden=hidden, n_heads=1, head_dim=64, n_experts=experts, top_k=top_k, moe_inter=width,
                            vocab=300, dtype=dtype, logit_scale=8.0 if dtype == "f32" else 1.0)
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
