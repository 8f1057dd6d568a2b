"""Steps at the token counts where the LM head takes half a task per wave (bf16, five, six and ten token tiles): the first and last
count of each, one and two token groups, vocabularies whose last half task, task or group of four tasks is not full, logits that
can be stored by four and that cannot, and row lists of undecided positions that fill fewer tiles than the step has."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun, OracleRun, bars_for, compare_logits, compare_step, make_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [300, 1090, 1102])      # 5, 18 and 18 tasks; half tasks of 12, 2 and 14 ids at the end
@pytest.mark.parametrize("n_seq,block", [(3, 43), (5, 32), (7, 23), (3, 64), (17, 17), (5, 64)])
def test_step_with_half_tasks_of_the_head(n_seq, block, vocab):
    check(n_seq, block, vocab, 320)


@pytest.mark.parametrize("hidden", [64, 128, 192, 256])       # fewer chunks of K than the loop keeps under way, as many, one more
@pytest.mark.parametrize("n_seq,block", [(5, 32), (5, 64)])
def test_half_tasks_of_a_short_contraction(n_seq, block, hidden):
    check(n_seq, block, 300, hidden)


def check(n_seq, block, vocab, hidden):
    cfg = di.configs.scaled(di.model_preset("tiny"), hidden=hidden, n_heads=2, head_dim=64, n_experts=8, moe_inter=64, vocab=vocab, dtype="bf16",
                            logit_scale=1.0)
    wl = di.Workload("half_head", cfg, n_seq, block, 2, 30, precommit=True, threshold=0.9, seed_index=160 + n_seq)
    cfg, w, inp = make_case(wl)
    cap = int(inp.prefix_len.max()) + 2 * block + 16
    ora = OracleRun(cfg, w, inp, cap)
    T = n_seq * block
    gpu = GpuRun(cfg, w, inp, T, cap)
    bars = bars_for(cfg)
    gpu.inject_prefix(ora.caches)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    got = gpu.step(wl.threshold)
    logits = gpu.logits(T).reshape(n_seq, block, vocab)
    routing = gpu.routing().reshape(cfg.n_layers, n_seq, block, cfg.top_k)
    for s in range(n_seq):
        ref, _ = ora.step_following(s, inp.block_tokens[s], int(inp.mask_bits[s]), int(inp.prefix_len[s]), wl.threshold, 0, routing[:, s], bars)
        compare_logits(ref["logits"], logits[s], bars)
        compare_step(ref, got["tokens"][s], got["mask"][s], got["conf"][s], got["argmax"][s], got["n_committed"][s],
                     inp.block_tokens[s], inp.mask_bits[s], wl.threshold, 0, bars, ref["logits"], logits[s])
    # the same rows through a list: every sequence but the first keeps three undecided positions, the others' entries stay as they are
    few = inp.mask_bits.copy()
    few[1:] = [1 | 1 << (block // 2) | 1 << (block - 1)] * (n_seq - 1)
    gpu.set_state(inp.block_tokens, few, inp.prefix_len)
    gpu.conf.fill_(-7.0)
    gpu.argmax.fill_(-7)
    listed = gpu.step(gpu.binding.Decode(wl.threshold, 0, 0, 0.0, 1))
    for s in range(n_seq):
        on = np.array([(int(few[s]) >> i) & 1 for i in range(block)], dtype=bool)
        assert np.array_equal(listed["conf"][s][on], got["conf"][s][on]) and np.array_equal(listed["argmax"][s][on], got["argmax"][s][on])
        assert (listed["conf"][s][~on] == -7).all() and (listed["argmax"][s][~on] == -7).all()
    gpu.close()


# lists that fill three to ten tiles: one token group of four, five and six tiles; two groups of 4 + 3, 4 + 4, 5 + 4 and 5 + 5
@pytest.mark.parametrize("n_seq,block,counts", [(5, 32, (96, 97, 100, 128, 129, 159)), (3, 64, (128, 129, 160, 161, 191)),
                                                (5, 64, (96, 128, 129, 160, 161, 192, 193, 224, 225, 256, 257, 288, 289, 319))])
def test_row_lists_of_every_number_of_tiles(n_seq, block, counts):
    cfg = di.configs.scaled(di.model_preset("tiny"), hidden=320, n_heads=2, head_dim=64, n_experts=8, moe_inter=64, vocab=1102, dtype="bf16",
                            logit_scale=1.0)
    cfg, w, inp = make_case(di.Workload("half_list", cfg, n_seq, block, 2, 30, threshold=0.9, seed_index=170 + n_seq))
    T, cap = n_seq * block, int(inp.prefix_len.max()) + 2 * block + 16
    gpu = GpuRun(cfg, w, inp, T, cap)
    gpu.ctx.kv.zero_()
    rng = np.random.default_rng(T)
    for n in counts:
        on = np.zeros(T, dtype=bool)
        on[::block] = True                                  # one position of every sequence, the others anywhere
        on[rng.permutation(np.flatnonzero(~on))[:n - n_seq]] = True
        on = on.reshape(n_seq, block)
        masks = np.array([sum(1 << int(i) for i in np.flatnonzero(row)) for row in on], dtype=np.uint64)
        gpu.set_state(inp.block_tokens, masks, inp.prefix_len)
        full = gpu.step(0.9)
        gpu.set_state(inp.block_tokens, masks, inp.prefix_len)
        gpu.conf.fill_(-7.0)
        gpu.argmax.fill_(-7)
        listed = gpu.step(gpu.binding.Decode(0.9, 0, 0, 0.0, 1))
        for key in ("conf", "argmax"):
            assert np.array_equal(listed[key][on], full[key][on]) and (listed[key][~on] == -7).all(), (n, key)
    gpu.close()
