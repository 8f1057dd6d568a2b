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


def model(dtype, n_seq, block, hidden, experts, top_k, width):
    """One layer whose attention adds nothing to rows of ones (1/rms is 1 but for epsilon); every other weight is zero."""
    cfg = di.configs.scaled(di.model_preset("tiny"), n_layers=1, hidden=hidden, n_heads=1, head_dim=64, n_experts=experts, top_k=top_k,
                            moe_inter=width, vocab=64, dtype=dtype, logit_scale=1.0)
    weights = di.make_weights(cfg, di.BASE_SEED)
    inp = di.make_workload_inputs(di.Workload("order", cfg, n_seq, block, 2, 10, threshold=2.0, seed_index=190))
    for name, a in weights["layers"][0].items():
        if name.startswith("w"):
            zeros(a)
        else:
            a[...] = 1
    put(dtype, weights["emb"], ..., 1.0)
    return cfg, weights, inp


def step(cfg, weights, inp, T):
    gpu = GpuRun(cfg, weights, inp, T, 128)
    gpu.ctx.kv.zero_()
    gpu.set_state(inp.block_tokens, inp.mask_bits, inp.prefix_len)
    gpu.step(2.0)
    hidden = gpu.ctx.debug_get(0, (T, cfg.hidden), gpu.torch.float32).cpu().numpy()
    routing = gpu.routing(T)[0]
    gpu.close()
    return hidden, routing


def router_case(dtype, n_seq, block, hidden, small, negative):
    """Expert 0's logit: BIG from feature 0, 0.75 from each of the features `small`, -BIG from feature `negative`; expert 1's is 1.
    Returns whether expert 0 was taken by every token, that is whether the small terms are left."""
    cfg, weights, inp = model(dtype, n_seq, block, hidden, 2, 1, 64)
    w = weights["layers"][0]["w_router"]
    put(dtype, w, (0, 0), BIG)
    for f in small:
        put(dtype, w, (0, f), 0.75)
    put(dtype, w, (0, negative), -BIG)
    put(dtype, w, (1, 5), 1.0)
    taken = step(cfg, weights, inp, n_seq * block)[1][:, 0]
    assert (taken == taken[0]).all()
    return taken[0] == 0


# features per chain of the contraction: eight waves of up to eight k-steps of sixteen features, the waves of several workgroups
# where that divides K
@pytest.mark.parametrize("n_seq,block", [(1, 1), (1, 11), (1, 32), (2, 16)])
@pytest.mark.parametrize("hidden,chain", [(2048, 128), (4096, 128), (3072, 128), (1024, 128), (512, 64), (1536, 192)])
def test_router_of_up_to_32_tokens_adds_along_its_chains(hidden, chain, n_seq, block):
    assert not router_case("bf16", n_seq, block, hidden, range(16, chain, 16), chain)
    assert router_case("bf16", n_seq, block, hidden, range(chain, 2 * chain, 16), 2 * chain)      # a chain of their own


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
    hidden, _ = step(cfg, weights, inp, T)
    y = 1 / (1 + np.exp(-1)) / 5
    ulp = np.spacing(np.float32(BIG * y))
    assert (hidden[:, 0] == 1).all()
    assert (np.abs(hidden[:, 1] - 1 - 8 * 0.5 * y) <= ulp).all()      # two sums with BIG * y in them, half an ulp each
    assert (hidden[:, 2:] == 1).all()
