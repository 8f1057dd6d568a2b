"""Orders of sums that a deep model's routing hangs on: where two experts tie, another order of the same float32 sum takes the other
one, and sixteen layers make a different row of it.  The operands here show the order: a large term, terms that a sum already
holding the large one rounds away, and the large one's negative, so that the result is zero if the small terms were added behind the
large one, and their sum (rounded) if they were added to each other first.  All are exact in the weights' type."""
import numpy as np
import pytest

import dinfer_inputs as di
from harness import GpuRun

pytestmark = pytest.mark.gpu

BIG = 2.0 ** 24          # a float32 sum of it and less than 1 is BIG, by rounding to nearest or towards zero


def zeros(a):
    a[...] = 0


def put(dtype, a, where, value):
    a[where] = np.float32(value) if dtype == "f32" else np.uint16(np.float32(value).view(np.uint32) >> 16)


def model(dtype, n_seq, block, hidden, experts, top_k, width, prefix=None, n_heads=1, vocab=64):
    """One layer whose attention adds nothing to rows of ones (1/rms is 1 but for epsilon); every other weight is zero."""
    cfg = di.configs.scaled(di.model_preset("tiny"), n_layers=1, hidden=hidden, n_heads=n_heads, head_dim=64, n_experts=experts, top_k=top_k,
                            moe_inter=width, vocab=vocab, dtype=dtype, logit_scale=1.0)
    weights = di.make_weights(cfg, di.BASE_SEED)
    inp = di.make_workload_inputs(di.Workload("order", cfg, n_seq, block, prefix or 2, prefix or 10, threshold=2.0, seed_index=190))
    for name, a in weights["layers"][0].items():
        if name.startswith("w"):
            zeros(a)
        else:
            a[...] = 1
    put(dtype, weights["emb"], ..., 1.0)
    return cfg, weights, inp


def step(cfg, weights, inp, T, max_pos=128, fill=None):
    gpu = GpuRun(cfg, weights, inp, T, max_pos)
    gpu.ctx.kv.zero_()
    if fill:
        fill(gpu)
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    gpu.step(2.0)
    hidden = gpu.ctx.debug_get(0, (T, cfg.hidden), gpu.torch.float32).cpu().numpy()
    routing = gpu.routing(T)[0]
    weights = gpu.ctx.debug_get(2, (cfg.n_layers, T, cfg.top_k), gpu.torch.float32).cpu().numpy()[0]
    gpu.close()
    return hidden, routing, weights


def router_case(dtype, n_seq, block, hidden, small, negative, n_heads=1):
    """Expert 0's logit: BIG from feature 0, 0.75 from each of the features `small`, -BIG from feature `negative`; expert 1's is 1.
    Returns whether expert 0 was taken by every token, that is whether the small terms are left."""
    cfg, weights, inp = model(dtype, n_seq, block, hidden, 2, 1, 64, n_heads=n_heads)
    w = weights["layers"][0]["w_router"]
    put(dtype, w, (0, 0), BIG)
    for f in small:
        put(dtype, w, (0, f), 0.75)
    put(dtype, w, (0, negative), -BIG)
    put(dtype, w, (1, 5), 1.0)
    taken = step(cfg, weights, inp, n_seq * block)[1][:, 0]
    assert (taken == taken[0]).all()
    return taken[0] == 0


def check_chains(hidden, chain, n_seq, block, n_heads=1):
    assert not router_case("bf16", n_seq, block, hidden, range(16, chain, 16), chain, n_heads)
    assert router_case("bf16", n_seq, block, hidden, range(chain, 2 * chain, 16), 2 * chain, n_heads)      # a chain of their own


# features per chain of the contraction: eight waves of up to eight k-steps of sixteen features, the waves of several workgroups
# where that divides K
@pytest.mark.parametrize("n_seq,block", [(1, 1), (1, 11), (1, 32), (2, 16)])
@pytest.mark.parametrize("hidden,chain", [(2048, 128), (4096, 128), (3072, 128), (1024, 128), (512, 64), (1536, 192)])
def test_router_of_up_to_32_tokens_adds_along_its_chains(hidden, chain, n_seq, block):
    check_chains(hidden, chain, n_seq, block)


# ... of four k-steps, with two token tiles
@pytest.mark.parametrize("n_seq,block", [(1, 33), (1, 64), (4, 16)])
@pytest.mark.parametrize("hidden,chain", [(2048, 64), (4096, 64), (1536, 64), (512, 64), (768, 96), (320, 48)])
def test_router_of_33_to_64_tokens_adds_along_its_chains(hidden, chain, n_seq, block):
    check_chains(hidden, chain, n_seq, block)


# ... an eighth of K (two heads: the output projection takes its dense form)
@pytest.mark.parametrize("n_seq,block", [(5, 13), (5, 32), (16, 33)])
@pytest.mark.parametrize("hidden,chain", [(2048, 256), (1024, 128), (768, 96), (320, 48)])
def test_router_of_many_tokens_adds_along_its_chains(hidden, chain, n_seq, block):
    check_chains(hidden, chain, n_seq, block, 2)


# With the test switch on, no part of a logit comes from another workgroup: one workgroup contracts all of K, an eighth per wave.
@pytest.mark.parametrize("n_seq,block", [(1, 1), (1, 32), (1, 33), (4, 16), (5, 13)])
@pytest.mark.parametrize("dtype,hidden,chain,kstep", [("f32", 512, 64, 8), ("f32", 2048, 256, 8), ("bf16", 2048, 256, 16)])
def test_single_slice_contracts_the_router_in_one_workgroup(dtype, hidden, chain, kstep, n_seq, block):
    from paper_2510_08666_amd import binding
    binding.debug_single_slice(True)
    try:
        assert not router_case(dtype, n_seq, block, hidden, range(kstep, chain, kstep), chain)
        assert router_case(dtype, n_seq, block, hidden, range(chain, 2 * chain, kstep), 2 * chain)
    finally:
        binding.debug_single_slice(False)


# 5 experts of 2048 are 80 groups of eight k-steps for 64 waves: two each in list order, the last 24 waves none
@pytest.mark.parametrize("n_seq,block", [(1, 1), (1, 32)])
def test_fused_down_projection_cuts_its_contraction_into_equal_shares(n_seq, block):
    T, group = n_seq * block, 128
    cfg, weights, inp = model("bf16", n_seq, block, 64, 5, 5, 2048)
    layer = weights["layers"][0]
    put("bf16", layer["w_gate"], (slice(None), slice(None), 0), 1.0)
    put("bf16", layer["w_up"], (slice(None), slice(None), 0), 1.0)
    # every element of the experts' intermediate rows is y = silu(1) / 5; BIG * y + 0.5 * y is BIG * y.  Features 0 and 1 of expert 0:
    # the small terms in the group behind the large one's, which is the same wave's, and in the one after it, the next wave's
    w = layer["w_down"]
    for feature, small in ((0, 1), (1, 2)):
        put("bf16", w, (0, feature, 0), BIG)
        put("bf16", w, (0, feature, slice(small * group, (small + 1) * group, 16)), 0.5)
        put("bf16", w, (0, feature, 4 * group), -BIG)
    hidden, _, _ = step(cfg, weights, inp, T)
    y = 1 / (1 + np.exp(-1)) / 5
    ulp = np.spacing(np.float32(BIG * y))
    assert (hidden[:, 0] == 1).all()
    assert (np.abs(hidden[:, 1] - 1 - 8 * 0.5 * y) <= ulp).all()      # two sums with BIG * y in them, half an ulp each
    assert (hidden[:, 2:] == 1).all()


# Sixteen splits of the keys, dealt by tiles of 32 to eight waves each: split p has keys 256 p on.  One key each in splits 0 to 7 has
# all of the split's weight, and one in split 8 a little more.  Splits 0 and 1 have values that cancel: each multiplied by its weight
# against the maximum of all, with a fused add, they leave the first one's rounding; added first and scaled then, nothing.
def test_attention_folds_its_splits_against_one_maximum():
    block, prefix, value = 5, 8187, 1.3984375 * 2.0 ** 20
    cfg, weights, inp = model("bf16", 1, block, 64, 2, 1, 64, prefix)
    layer = weights["layers"][0]
    put("bf16", layer["wq"], (31, 0), 16.0)      # the pair of features that positions turn least
    put("bf16", layer["wo"], (0, 0), 1.0)

    def fill(gpu):
        kv = gpu.torch.zeros((2, prefix, cfg.n_heads * cfg.head_dim), dtype=gpu.torch.float32, device=gpu.dev)
        kv[0, 0:8 * 256:256, 31] = 100.0
        kv[0, 8 * 256, 31] = 100.5
        kv[1, 0, 0], kv[1, 256, 0] = value, -value
        gpu.ctx.kv_write(0, gpu.page_table[0], 0, kv[0], kv[1])

    hidden, _, _ = step(cfg, weights, inp, block, prefix + 2 * block, fill)
    off = np.abs(hidden[:, 0] - 1)
    assert off.any() and (off <= value * 2.0 ** -24).all()
    assert (hidden[:, 1:] == 1).all()


# Rows whose squares have more than 24 bits, in features that a lane of the output projection holds together: which of a pair's two squares
# is rounded by itself is the same in split-K (63 tokens) and in workgroups of one and of two token tiles (72, 522).
@pytest.mark.parametrize("more", [8, 58])
def test_row_statistics_round_alike_in_every_form(more):
    got = []
    for n_seq in (7, more):
        cfg, weights, inp = model("bf16", n_seq, 9, 4096, 2, 2, 64, n_heads=2)
        layer, on = weights["layers"][0], list(range(8)) + list(range(32, 40))
        put("bf16", weights["emb"], ..., 0.0)
        for f in on:
            weights["emb"][:, f] = np.random.default_rng(f).standard_normal(cfg.vocab).astype(np.float32).view(np.uint32) >> 16
        inp.block_tokens[...] = np.arange(n_seq * 9).reshape(n_seq, 9) % cfg.vocab
        put("bf16", layer["wo"], (on, on), 1.3671875)
        put("bf16", layer["w_router"], (0, 0), 0.5)

        def fill(gpu):
            values = np.random.default_rng(7).standard_normal((more, cfg.n_heads * cfg.head_dim))
            for s in range(n_seq):
                n = int(inp.prefix_len[s])
                k = gpu.torch.zeros((n, values.shape[1]), dtype=gpu.torch.float32, device=gpu.dev)
                v = gpu.torch.from_numpy(values[s]).to(gpu.torch.bfloat16).float().to(gpu.dev).expand(n, -1).contiguous()
                gpu.ctx.kv_write(0, gpu.page_table[s], 0, k, v)

        got.append([a[:63] for a in step(cfg, weights, inp, 9 * n_seq, fill=fill)])
    for a, b in zip(*got):
        assert np.array_equal(a, b)
    assert len(np.unique(got[0][2])) > 63


# The LM head takes half a task per wave at five, six and ten token tiles and whole tasks at three: a lane's sum of exponentials is
# over the 32 ids that it has of a whole task, in their order, either way.  (The layer adds nothing, so the rows are the same.)
@pytest.mark.parametrize("n_seq", [5, 6, 10])
def test_sums_of_exponentials_run_on_from_half_to_half(n_seq):
    got = []
    for n in (3, n_seq):
        cfg, weights, inp = model("bf16", n, 32, 128, 2, 1, 64, vocab=1102)
        weights["emb"][...] = di.make_weights(cfg, di.BASE_SEED + 3)["emb"]
        inp.block_tokens[...] = np.arange(n * 32).reshape(n, 32)
        gpu = GpuRun(cfg, weights, inp, n * 32, 128)
        gpu.ctx.kv.zero_()
        gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
        state = gpu.step(2.0)
        got.append((state["conf"][:3], state["argmax"][:3]))
        gpu.close()
    assert len(np.unique(got[0][0])) > 90
    assert np.array_equal(got[0][0], got[1][0]) and np.array_equal(got[0][1], got[1][1])
