"""The merge of the LM head's softmax partials (one per 64 ids above 64 tokens, 256 of them a round of its workgroup, 16 rounds
in flight) at one round, a little more, sixteen rounds and a few partials beyond, against the softmax of the step's own
logits in 64 bits."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("vocab", [16384, 16385, 262144, 262145])
def test_confidence_over_rounds(vocab, dtype):
    n_seq, block = 2, 35
    cfg = di.configs.scaled(di.model_preset("tiny"), n_layers=1, hidden=64, n_heads=1, moe_inter=64, vocab=vocab, dtype=dtype,
                            logit_scale=8.0)
    wl = di.Workload("merge", cfg, n_seq, block, 5, 40, threshold=2.0, seed_index=150)
    cfg, w, inp = make_case(wl)
    gpu = GpuRun(cfg, w, inp, n_seq * block, int(inp.prefix_len.max()) + block + 16)
    gpu.ctx.kv.zero_()
    ids = np.random.default_rng(vocab).integers(0, vocab - 1, (n_seq, block)).astype(np.int32)
    gpu.set_state(ids, np.full(n_seq, 2 ** block - 1, dtype=np.uint64), inp.prefix_len)
    got = gpu.step(2.0)
    logits = gpu.ctx.debug_logits(n_seq * block)
    assert np.array_equal(got["argmax"].reshape(-1), np.argmax(logits.cpu().numpy(), axis=1))
    want = gpu.torch.softmax(logits.double(), dim=-1).max(dim=-1).values.cpu().numpy()
    # float32 sums of 64 terms, then a tree over the partials, of exponentials good to about 2e-6: the bound is ten times that
    assert np.abs(got["conf"].reshape(-1) / want - 1).max() < 2e-5
    gpu.close()
