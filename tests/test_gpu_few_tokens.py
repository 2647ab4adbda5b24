"""Experts with few tokens: the tiles that the grouped FFN streams (64 rows, 32 or 64 weight rows per
workgroup, the sum over K split between wavefronts), at the edges of their row blocks, for the smallest
and odd K ranges of a wavefront, alone in a launch and beside larger tiles; in one wave and in many."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import assert_close, bf16_tensor_to_f32, make_runner, oracle_layer, say
from paper_2310_18859_amd.runner import MoERunner
from workloads import Workload, gen_gate, gen_x

pytestmark = pytest.mark.gpu

EDGES = [1, 2, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64]
SEVERAL = [65, 130, 1, 64, 129]                        # experts of several streamed tiles
# 50 experts of 1..45 tokens beside six of 65..250: too few to be streamed beside those, all are walked
BESIDE = [1 + (7 * i) % 45 for i in range(50)] + [65, 96, 127, 128, 129, 250]
# as many more as fill the chip beside the larger tiles of a layer of 256 columns
BESIDE_MANY = [1 + (7 * i) % 45 for i in range(130)] + [65, 96, 127, 128, 129, 250]
FEWER = [1, 64, 17, 31, 32, 33]
# more than ten tokens each and no larger tiles: streamed where they leave most of the chip idle or fill it
ALONE = [12 + (5 * i) % 20 for i in range(60)]
ALONE_MANY = [12 + (5 * i) % 20 for i in range(70)]

# the lines between streamed and walked experts beside larger tiles: 20, 28 or 36 tokens, or none, by each GEMM
LINES = [19, 20, 21, 27, 28, 29, 35, 36, 37, 1, 33, 32]


def lines(times, larger):
    return LINES * times + [129 + 7 * i % 300 for i in range(larger)]


def ids_with_counts(counts, seed):
    ids = np.repeat(np.arange(len(counts), dtype=np.int32), counts)
    return np.random.default_rng(seed).permutation(ids).astype(np.int32)


def forward(r, x_bits, ids, alpha):
    plan = r.ctx.moe_plan(0, ids)
    x, i, a, y = r.to_device(x_bits, ids, alpha)
    y.fill_(7.0)                                        # every row must be overwritten
    torch.cuda.synchronize()
    r.ctx.moe_layer_forward(plan, x, i, a, y, r.workspace, r.compute, r.copy)
    r.sync()
    return plan, y


ALL = 2**31 - 1
# name, counts, d, F, and the most tokens of a streamed expert in either GEMM (test_tile_rule_host.py looks whether it is so)
CASES = [
    ("edges", EDGES, 128, 128, (ALL, ALL)),             # one step of 32 K values per wavefront
    ("edges", EDGES, 384, 640, (ALL, ALL)),             # 3 and 5 steps: less than are loaded ahead
    ("edges", EDGES, 768, 3072, (ALL, ALL)),
    ("several-tiles", SEVERAL, 256, 896, (ALL, ALL)),   # 7 steps
    ("beside-larger", BESIDE, 256, 512, (0, 0)),
    ("beside-larger", BESIDE, 128, 896, (0, 0)),
    ("beside-many", BESIDE_MANY, 256, 512, (28, 64)),
    ("beside-many", BESIDE_MANY, 384, 640, (28, 0)),
    ("alone", ALONE, 256, 512, (64, 64)),
    ("alone", ALONE_MANY, 512, 896, (64, 64)),
    ("alone-walked", ALONE_MANY, 384, 256, (0, 0)),     # between the two
    ("lines-many", lines(6, 2), 384, 640, (28, 64)),
    ("lines-many", lines(8, 2), 384, 1536, (20, 64)),
    ("lines-many", lines(10, 2), 512, 896, (28, 0)),
    # layers whose larger experts weigh more
    ("lines-round", lines(2, 8), 512, 2048, (0, 0)),
    ("lines-round", lines(3, 30), 384, 768, (36, 0)),
    ("lines-round", lines(5, 30), 512, 896, (0, 20)),
    # every length of a sum up to two rounds of the steps that are loaded ahead, and one more
    ("lengths", FEWER, 512, 1024, (ALL, ALL)),          # 4 and 8 steps
    ("lengths", FEWER, 1152, 1280, (ALL, ALL)),         # 9 and 10
    ("lengths", FEWER, 1408, 1536, (ALL, ALL)),         # 11 and 12
    ("lengths", FEWER, 256, 1664, (ALL, ALL)),          # 2 and 13
    # more layers on either side of the lines
    ("lines-many", lines(10, 4), 512, 1024, (20, 20)),
    ("lines-many", lines(4, 2), 896, 512, (64, 28)),
    ("lines-round", lines(5, 10), 384, 768, (20, 0)),   # beside tiles of 64 rows
    ("lines-round", lines(5, 20), 512, 896, (28, 0)),
    ("lines-round", lines(2, 30), 896, 512, (0, 36)),
    ("lines-many", lines(6, 4), 896, 512, (36, 28)),
    ("lines-round", lines(4, 35), 512, 896, (0, 28)),
    ("lines-part", [64, 65, 63] * 2 + lines(6, 1), 512, 896, (28, 64)),
    ("lines-part", [64, 65, 63] * 2 + lines(4, 1), 896, 512, (64, 0)),
]


@pytest.mark.parametrize("name,counts,d,F", [c[:4] for c in CASES])
def test_few_token_experts(name, counts, d, F):
    T, E = sum(counts), len(counts)
    say(f"few-token experts: {name} E={E} T={T} d={d} F={F}")
    wl = Workload(600 + len(counts), name, 1, E, d, F, T, None, E, E)
    x_bits, ids, alpha = gen_x(wl, 0), ids_with_counts(counts, d + F), gen_gate(wl, 0)
    r = make_runner(wl)
    ref = oracle_layer(wl, r, 0, x_bits, ids, alpha)
    out = {}
    for fused in (False, True):
        r.ctx.set_fusion(fused)
        _, y = forward(r, x_bits, ids, alpha)
        assert_close(bf16_tensor_to_f32(y), ref, f"{name} fused={fused}")
        out[fused] = y.view(torch.uint16).cpu().numpy()
    assert np.array_equal(out[False], out[True])
    # cut into waves of at most five experts: the same sums in the same order
    rw = MoERunner(1, E, d, F, 10 if E > 10 else E, 5, T)
    rw.host_weights = r.host_weights
    rw.ctx.bind_host_weights([r.host_weights.data_ptr() + e * rw.expert_bytes for e in range(E)], keep=r.host_weights)
    plan, y = forward(rw, x_bits, ids, alpha)
    assert plan.n_waves >= (E + 4) // 5
    assert np.array_equal(y.view(torch.uint16).cpu().numpy(), out[True])
    rw.close()
    r.close()


def test_few_token_experts_two_per_token():
    E, d, F, k = 9, 256, 384, 2
    tokens = 70
    say(f"few-token experts: {k} per token, E={E}")
    wl = Workload(640, "few-topk", 1, E, d, F, tokens * k, None, E, E)
    rng = np.random.default_rng(3)
    x_bits, alpha = gen_x(wl, 0, tokens), gen_gate(wl, 0, tokens * k)
    ids = rng.integers(0, E, tokens * k).astype(np.int32)
    r = make_runner(wl)
    r.ctx.set_top_k(k)
    hw = r.host_weights.numpy()
    ref = oracle.moe_forward_topk(x_bits, ids.reshape(tokens, k), alpha.reshape(tokens, k), [hw[e] for e in range(E)], d, F)
    for fused in (False, True):
        r.ctx.set_fusion(fused)
        _, y = forward(r, x_bits, ids, alpha)
        assert_close(bf16_tensor_to_f32(y), ref, f"top-{k} fused={fused}")
    r.close()
