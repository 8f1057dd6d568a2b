"""Rows that are not numbers (a broken embedding row, a caller's expected embedding gone wrong): the sequence that holds
them has no result, the others keep theirs, and nothing is indexed by what comes out of such a row."""
import numpy as np
import pytest

import dinfer_inputs as di
import oracle
from harness import GpuRun, bars_for, make_case

pytestmark = pytest.mark.gpu


# token counts of the router's forms: one and two token tiles, whose pairs the expert kernels sort, and the permutation over groups
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n_seq,block", [(2, 16), (2, 32), (3, 40)])
def test_sequence_of_not_a_number(n_seq, block, dtype):
    cfg = di.configs.scaled(di.model_preset("tiny"), dtype=dtype, logit_scale=8.0 if dtype == "f32" else 1.0)
    wl = di.Workload("nan", cfg, n_seq, block, 20, 60, threshold=2.0, seed_index=95)
    cfg, w, inp = make_case(wl)
    bad = 17
    w["emb"][bad] = np.float32(np.nan) if dtype == "f32" else np.uint16(0x7FC0)
    gpu = GpuRun(cfg, w, inp, n_seq * block, 128)
    gpu.ctx.kv.zero_()
    tokens, masks = inp.block_tokens.copy(), inp.mask_bits.copy()
    masks[0] &= ~np.uint64(1 << 3)
    tokens[0, 3] = bad + 1
    for s in range(n_seq):
        assert not (tokens[s] == bad).any()
    gpu.set_state(tokens, masks, inp.prefix_len)
    want = gpu.step(2.0)
    z_want = gpu.logits(n_seq * block).reshape(n_seq, block, -1)
    tokens[0, 3] = bad
    gpu.set_state(tokens, masks, inp.prefix_len)
    got = gpu.step(2.0)
    z_got = gpu.logits(n_seq * block).reshape(n_seq, block, -1)
    routing = gpu.routing()
    assert routing.min() >= 0 and routing.max() < cfg.n_experts
    assert (np.diff(np.sort(routing, axis=-1), axis=-1) > 0).all()
    n_pairs = n_seq * block * cfg.top_k
    tables = [gpu.ctx.debug_get(f, (n,), gpu.torch.int32).cpu().numpy() for f, n in ((3, cfg.n_experts), (4, cfg.n_experts + 1), (5, n_pairs))]
    for table, ref in zip(tables, oracle.permutation(routing[-1].reshape(-1), cfg.n_experts)):
        assert np.array_equal(table, ref)
    assert np.isnan(z_got[0]).all()
    # the other sequences: their rows sit elsewhere among the experts' rows now, and the split of the fused down projection
    # follows the experts that have rows, so float32 sums may run in another order
    rel = bars_for(cfg).logit_rel
    for s in range(1, n_seq):
        assert np.abs(z_got[s] - z_want[s]).max() <= rel * np.abs(z_want[s]).max()
        assert np.array_equal(got["tokens"][s], want["tokens"][s]) and got["n_committed"][s] == want["n_committed"][s] == 1
    gpu.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_credit_lists_survive_not_a_number(dtype):
    """A credit step over a sequence of NaN leaves list entries without an id of the vocabulary; the next step over the same
    lists, with numbers again, gives what it gives with lists that never saw them."""
    cfg = di.configs.scaled(di.model_preset("tiny"), dtype=dtype, logit_scale=8.0 if dtype == "f32" else 1.0)
    wl = di.Workload("nan_credit", cfg, 2, 16, 20, 60, threshold=2.0, seed_index=96)
    cfg, w, inp = make_case(wl)
    bad = 17
    w["emb"][bad] = np.float32(np.nan) if dtype == "f32" else np.uint16(0x7FC0)
    gpu = GpuRun(cfg, w, inp, 32, 128)
    gpu.ctx.kv.zero_()
    masks = inp.mask_bits.copy()
    masks[0] &= ~np.uint64(1 << 3)

    def step(credit, first):
        tokens = inp.block_tokens.copy()
        tokens[0, 3] = first
        gpu.set_state(tokens, masks, inp.prefix_len)
        return gpu.step_credit(credit, 2.0, 0.5, 0.9, 0.7)

    lists = gpu.credit_state()
    step(lists, bad)
    ids = lists["ids"].cpu().numpy()[0, :, 0]
    assert not ((ids[np.arange(16) != 3] >= 0) & (ids[np.arange(16) != 3] < cfg.vocab)).any()
    got = step(lists, bad + 1)
    assert np.isfinite(got["conf"]).all() and (got["argmax"] >= 0).all() and (got["argmax"] < cfg.vocab).all()
    want = step(gpu.credit_state(), bad + 1)
    # sequence 0: the same single candidate with the same credit; sequence 1 has credit from the first step already
    assert np.array_equal(got["argmax"][0], want["argmax"][0])
    assert np.allclose(got["conf"][0], want["conf"][0], rtol=1e-5)
    gpu.close()
