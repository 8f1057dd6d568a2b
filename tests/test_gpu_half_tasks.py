"""Steps of up to 32 tokens whose QKV projection takes half a task per workgroup (bf16, 64 to 128 tasks of 64 features, K of
1024 or 2048 cut over eight waves): both K shares, the fewest and nearly the most tasks, one token, ragged and full tiles."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, kv_close, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,n_heads", [(1024, 11), (2048, 21)])       # 66 and 126 tasks
@pytest.mark.parametrize("n_seq,block", [(1, 1), (3, 9), (1, 32)])
def test_step_with_half_tasks(hidden, n_heads, n_seq, block):
    cfg = di.configs.scaled(di.model_preset("tiny"), hidden=hidden, n_heads=n_heads, head_dim=128, n_experts=8, moe_inter=64, vocab=500,
                            dtype="bf16", logit_scale=1.0)
    wl = di.Workload("half", cfg, n_seq, block, 3, 40, threshold=0.9, seed_index=110 + block)
    cfg, w, inp = make_case(wl)
    cap = int(inp.prefix_len.max()) + 2 * block + 16
    ora = OracleRun(cfg, w, inp, cap)
    gpu = GpuRun(cfg, w, inp, n_seq * block, cap)
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    got = gpu.step(wl.threshold)
    logits = gpu.logits(n_seq * block).reshape(n_seq, block, cfg.vocab)
    routing = gpu.routing().reshape(cfg.n_layers, n_seq, block, cfg.top_k)
    for s in range(n_seq):
        n = int(inp.prefix_len[s])
        ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), n, wl.threshold, 0, routing[:, s], bars)
        compare_logits(ref["logits"], logits[s], bars)
        compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                     inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"], logits[s])
        kc, vc = ora.caches[s]
        for l in range(cfg.n_layers):
            k, v = gpu.read_kv(s, l, n, block)
            assert kv_close(k, kc[l, n:n + block], bars) and kv_close(v, vc[l, n:n + block], bars), (s, l)
    gpu.close()
