"""Steps over vocabularies at which the LM head deals its tasks out differently, with ragged last groups and ids, against
the oracle."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, make_case

pytestmark = pytest.mark.gpu


# (vocabulary, sequences, block length).  262000 ids are 4094 tasks: 1024 groups of four, exactly two rounds of the chip,
# the last group with two tasks.  131500 ids: 514 groups, two of them beyond a round and handed out task by task.
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vocab,n_seq,block", [(262000, 1, 48), (131500, 3, 16)])
def test_step_over_vocabulary(vocab, n_seq, block, dtype):
    tiny = di.model_preset("tiny")
    cfg = di.configs.scaled(tiny, n_layers=1, hidden=128, n_heads=2, moe_inter=64, vocab=vocab, dtype=dtype,
                            logit_scale=8.0 if dtype == "f32" else 1.0)
    wl = di.Workload("vocabulary", cfg, n_seq, block, 20, 40, precommit=True, threshold=0.9, seed_index=90)
    cfg, w, inp = make_case(wl)
    ora = OracleRun(cfg, w, inp, 128)
    gpu = GpuRun(cfg, w, inp, n_seq * block, 128)
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    got = gpu.step(wl.threshold)
    logits = gpu.logits(n_seq * block).reshape(n_seq, block, vocab)
    routing = gpu.routing().reshape(cfg.n_layers, n_seq, block, cfg.top_k)
    for s in range(n_seq):
        ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), int(inp.prefix_len[s]), wl.threshold, 0,
                                    routing[:, s], bars)
        compare_logits(ref["logits"], logits[s], bars)
        compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                     inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"], logits[s])
    gpu.close()
