"""The logits hook behind a forward without an LM head (refresh of a block), which does not leave what the head of more than 64
bf16 tokens reads: they are those of that forward's rows, not of an earlier step's."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_seq,block", [(2, 32), (5, 13), (9, 60)])
def test_logits_behind_a_refresh(n_seq, block, dtype):
    tiny = di.model_preset("tiny")
    cfg = di.configs.scaled(tiny, vocab=1100, dtype=dtype, logit_scale=1.0)
    wl = di.Workload("headless", cfg, n_seq, block, 3, 70, threshold=0.9, seed_index=140 + n_seq)
    cfg, w, inp = make_case(wl)
    gpu = GpuRun(cfg, w, inp, n_seq * block, int(inp.prefix_len.max()) + 2 * block + 16)
    gpu.ctx.kv.zero_()
    ids = [np.random.default_rng(i).integers(0, cfg.vocab - 1, inp.block_tokens.shape).astype(np.int32) for i in (1, 2)]
    none = np.zeros(n_seq, dtype=np.uint64)

    def step(tokens):
        gpu.set_state(tokens, none, inp.prefix_len)
        gpu.step(wl.threshold)
        return gpu.logits(n_seq * block)

    want, other = step(ids[0]), step(ids[1])
    gpu.set_state(ids[0], none, inp.prefix_len)
    gpu.refresh()                      # the same forward as the first step
    assert np.array_equal(gpu.logits(n_seq * block), want) and not np.array_equal(want, other)
    gpu.close()
