"""Steps behind cached prefixes at the edges of attention's splits over the keys (32 keys a tile, up to 24 tiles one split, then
one per 16, at most 16): sequences of every number of splits side by side, ragged last tiles, maxima that lie in one split."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, kv_close, make_case

pytestmark = pytest.mark.gpu

BLOCK = 5
# keys = prefix + block.  Splits 1, 2, 2, 3 | 1, 4, 5, 5 | 8, 9, 9, 16 | 16, 1
PREFIXES = [[763, 764, 1019, 1020], [11, 2043, 2044, 2555], [4091, 4092, 4589, 8187], [8300, 1]]


@pytest.mark.parametrize("dtype,head_dim", [("f32", 64), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("lens", PREFIXES)
def test_step_behind_split_prefixes(lens, dtype, head_dim):
    cfg = di.configs.scaled(di.model_preset("tiny"), hidden=128, n_heads=2, head_dim=head_dim, n_experts=8, moe_inter=64, vocab=500,
                            dtype=dtype, logit_scale=8.0 if dtype == "f32" else 1.0)
    wl = di.Workload("splits", cfg, len(lens), BLOCK, 0, 0, threshold=0.9, seed_index=130)
    cfg, w, inp = make_case(wl, room=max(lens) + BLOCK)
    inp.prefix_len = np.array(lens, dtype=np.int32)
    ora = OracleRun(cfg, w, inp, max(lens) + BLOCK)
    for s, n in enumerate(lens):
        kc, vc = ora.caches[s]
        kc[:, :n], vc[:, :n] = di.synthetic_prefix_kv(cfg, inp.seed, s, n, peaked=4)
    gpu = GpuRun(cfg, w, inp, len(lens) * BLOCK, max(lens) + BLOCK + 16)
    gpu.ctx.kv.fill_(0xFF)           # not-a-numbers in the slots past a sequence's end must not matter
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    got = gpu.step(wl.threshold)
    logits = gpu.logits(len(lens) * BLOCK).reshape(len(lens), BLOCK, cfg.vocab)
    routing = gpu.routing().reshape(cfg.n_layers, len(lens), BLOCK, cfg.top_k)
    for s, n in enumerate(lens):
        ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), n, wl.threshold, 0, routing[:, s], bars)
        compare_logits(ref["logits"], logits[s], bars)
        compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                     inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"])
        kc, vc = ora.caches[s]
        for l in range(cfg.n_layers):
            k, v = gpu.read_kv(s, l, n, BLOCK)
            assert kv_close(k, kc[l, n:n + BLOCK], bars) and kv_close(v, vc[l, n:n + BLOCK], bars), (s, l)
    gpu.close()
