"""Steps of up to 64 tokens over models with more expert and vocabulary tasks than compute units, where the expert GEMMs and
the LM head take tasks whole, one per wave: odd task counts (the last workgroup has waves without a task), ids that fill
neither the last tile nor a vector store, one and two token tiles."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, make_case

pytestmark = pytest.mark.gpu


# 64 experts of width 192 over hidden 320: 6 and 5 tasks each, 384 and 320 in all; 16550 ids: 259 tasks
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_seq,block", [(1, 1), (1, 20), (2, 16), (1, 33), (3, 16), (1, 64)])
def test_step_with_whole_tasks(n_seq, block, dtype):
    cfg = di.configs.scaled(di.model_preset("tiny"), hidden=320, n_heads=2, head_dim=128, n_experts=64, top_k=8, moe_inter=192,
                            vocab=16550, dtype=dtype, logit_scale=8.0 if dtype == "f32" else 1.0)
    wl = di.Workload("whole", cfg, n_seq, block, 10, 60, precommit=block > 1, threshold=0.9, seed_index=80 + n_seq)
    cfg, w, inp = make_case(wl)
    ora = OracleRun(cfg, w, inp, 160)
    gpu = GpuRun(cfg, w, inp, n_seq * block, 160)
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    # one workgroup per sum: up to 32 tokens the down projection then takes the form that larger steps always take
    for single in (False, True):
        gpu.binding.debug_single_slice(single)
        try:
            gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
            got = gpu.step(wl.threshold)
            logits = gpu.logits(n_seq * block).reshape(n_seq, block, cfg.vocab)
            routing = gpu.routing().reshape(cfg.n_layers, n_seq, block, cfg.top_k)
        finally:
            gpu.binding.debug_single_slice(False)
        for s in range(n_seq):
            kc, vc = ora.caches[s]
            keep = kc.copy(), vc.copy()
            ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), int(inp.prefix_len[s]), wl.threshold, 0,
                                        routing[:, s], bars)
            kc[...], vc[...] = keep
            compare_logits(ref["logits"], logits[s], bars)
            compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                         inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"], logits[s])
    gpu.close()
