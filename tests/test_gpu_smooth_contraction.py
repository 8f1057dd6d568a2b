"""The expected-embedding contraction of the smoothing step at the sizes where its form changes (one, two and four token
tiles, one and several token groups, one slice, partial sums in place of the logits and in the workspace, a vocabulary
of no particular multiple),
against softmax(logits) . W_emb in 64 bits over the logits the same step produced."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_seq,block,vocab,hidden", [(1, 1, 1001, 256), (1, 32, 5000, 320), (3, 11, 4096, 256),
                                                      (2, 32, 2051, 128), (5, 13, 4096, 256), (4, 32, 1030, 64),
                                                      (3, 43, 4095, 192), (8, 40, 3000, 256), (2, 20, 100, 256),
                                                      (2, 20, 130, 1024), (3, 43, 700, 512), (20, 64, 4096, 1024),
                                                      (20, 60, 1030, 4096)])
def test_expected_embedding(n_seq, block, vocab, hidden, dtype):
    tiny = di.model_preset("tiny")
    cfg = di.configs.scaled(tiny, n_layers=1, hidden=hidden, vocab=vocab, dtype=dtype, logit_scale=4.0)
    wl = di.Workload("contraction", cfg, n_seq, block, 5, 40, precommit=True, threshold=2.0, seed_index=60 + n_seq)
    cfg, w, inp = make_case(wl)
    gpu = GpuRun(cfg, w, inp, n_seq * block, int(inp.prefix_len.max()) + block + 16)
    torch = gpu.torch
    gpu.ctx.kv.zero_()
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    sm = gpu.smooth_state()
    before = torch.randn_like(sm["delta"]) * 0.01
    sm["delta"].copy_(before)
    gpu.step_smooth(sm, 0.0, 2.0)
    p = torch.softmax(gpu.ctx.debug_logits(n_seq * block).double(), dim=-1)
    emb = w["emb"] if dtype == "f32" else di.bf16_to_f32(w["emb"])
    want = (p @ torch.from_numpy(np.asarray(emb)).to(gpu.dev).double()).view(n_seq, block, hidden)
    masked = torch.tensor([[(int(m) >> i) & 1 for i in range(block)] for m in inp.mask_bits], device=gpu.dev).bool()
    assert torch.equal(sm["delta"][~masked], before[~masked])
    # float32 sums of up to 5000 terms in another order, probabilities with 16 (bf16 hi + lo) or 24 bits and a hardware
    # exponential good to about 2e-6: a few 1e-6 of the row's norm; the bound is ten times that
    err = (sm["delta"].double() - want)[masked].norm(dim=-1) / want[masked].norm(dim=-1)
    assert float(err.max()) < 4e-5, float(err.max())
    gpu.close()
