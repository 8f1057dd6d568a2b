"""Prompt prefill where attention takes its many-rows form (bf16, at least 256 workgroups of four query tiles): prompt
lengths at the edges of its key turns (64 keys), query tiles (32) and groups (128), one prompt of a single turn, against
the oracle."""
from dataclasses import replace

import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, OracleRun, bars_for, kv_close, make_case

pytestmark = pytest.mark.gpu


# The last one takes attention in its other form and the output projection (hidden 4096) over eight tasks and four token
# tiles at once, as the others do the QKV projection.
@pytest.mark.parametrize("n_heads,head_dim,lens", [(32, 64, [385, 416, 447, 97]), (32, 128, [384, 353, 129, 200]),
                                                   (64, 64, [512, 97]), (64, 64, [500, 40]), (1, 128, [1057])])
def test_prefill_rows_form(n_heads, head_dim, lens):
    tiny = di.model_preset("tiny")
    cfg = di.configs.scaled(tiny, hidden=4096 if n_heads == 1 else 128, n_heads=n_heads, head_dim=head_dim, n_experts=8, moe_inter=64, vocab=500,
                            dtype="bf16", logit_scale=1.0)
    wl = di.Workload("prompts", cfg, len(lens), 1, 0, 0, threshold=0.9, seed_index=70)
    cfg, w, inp = make_case(wl, room=max(lens))
    inp.prefix_tokens = [np.random.default_rng([n, i]).integers(0, cfg.vocab - 1, n).astype(np.int32) for i, n in enumerate(lens)]
    inp.prefix_len = np.array(lens, dtype=np.int32)
    ora = OracleRun(cfg, w, replace(inp, prefix_tokens=[[] for _ in lens]), max(lens))
    gpu = GpuRun(cfg, w, inp, sum(lens), max(lens) + 16)
    bars = bars_for(cfg)
    # whatever the pool held before must not matter, not-a-numbers in the slots past a prompt's end included
    gpu.ctx.kv.fill_(0xFF)
    gpu.prefill()
    routing = gpu.routing(sum(lens))
    at = 0
    for s, n in enumerate(lens):
        ora.forward_following(s, inp.prefix_tokens[s], 0, routing[:, at:at + n], bars)
        at += n
        kc, vc = ora.caches[s]
        for l in range(cfg.n_layers):
            k, v = gpu.read_kv(s, l, 0, n)
            assert kv_close(k, kc[l, :n], bars) and kv_close(v, vc[l, :n], bars), (s, l)
    gpu.close()
