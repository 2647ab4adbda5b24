"""Where the grouped GEMM's walked tiles write: every row of y and nothing around it, with tiles that end one row before,
at and behind a block or tile edge, with y and x at any element's address, with every way the results leave (scattered,
and row by row where the gather and combine passes are kernels of their own)."""
import numpy as np
import pytest
import torch

from gpu_util import assert_close, bf16_tensor_to_f32, make_runner, oracle_layer
from workloads import Workload, gen_gate, gen_x

pytestmark = pytest.mark.gpu

EDGES = [700, 129, 128, 127, 97, 96, 65, 33, 32, 31, 1]     # 128-row tiles: 28 tiles of 64 rows, so none is streamed
SMALL = [64] * 20 + [63, 33, 32, 31, 1]                     # 64-row tiles
# So many experts of one tile that their weights, and the results with them, are streamed past L2's replacement (from 128
# MiB on): narrow tiles for 384 or 1152 columns and wide ones for 1536, for 64-row tiles also narrow ones that run four K-steps
# ahead (512 x 1024) and two (384 x 1152).
MANY_TALL = [300, 129] + [128, 127, 97, 96, 95, 66, 65] * 21 + [64, 33, 32, 31, 1]
MANY_SMALL = [130, 65] + [64, 63, 62, 34, 33] * 33 + [32, 31, 1]


def test_many_experts_are_past_the_rule():
    """... of launches whose single-tile weights are read once, for both tile heights."""
    for counts, rows, d, F in ((MANY_TALL, 128, 384, 1536), (MANY_SMALL, 64, 512, 1024), (MANY_SMALL, 64, 384, 1536),
                               (MANY_SMALL, 64, 384, 1152)):
        assert sum(n <= rows for n in counts) * d * F * 2 > 128 << 20 and len(counts) <= 255
        t64, t128 = (sum(-(-n // t) for n in counts) for t in (64, 128))
        assert (5 * t64 <= 6 * t128) == (rows == 64) and sum(n for n in counts if n <= 64) > 32 * sum(n <= 64 for n in counts)


@pytest.mark.parametrize("counts,d,F,shift,fused,k", [
    (EDGES, 256, 512, 0, True, 1), (EDGES, 256, 512, 1, True, 1), (EDGES, 384, 128, 4, True, 1),
    (EDGES, 256, 512, 0, False, 1), (EDGES + [2], 256, 512, 3, True, 3), (SMALL, 256, 512, 1, True, 1),
    (SMALL, 128, 384, 0, True, 1),
    (MANY_TALL, 384, 1536, 0, True, 1), (MANY_TALL, 1536, 384, 1, True, 1), (MANY_TALL, 384, 1536, 3, False, 1),
    (MANY_SMALL, 512, 1024, 0, True, 1), (MANY_SMALL, 1536, 384, 1, True, 1), (MANY_SMALL, 384, 1152, 5, True, 1),
    (MANY_SMALL, 512, 1024, 1, False, 1), (MANY_SMALL + [3], 384, 1536, 2, True, 3),
])
def test_results_and_nothing_else(counts, d, F, shift, fused, k):
    E, T = len(counts), sum(counts) // k * k
    wl = Workload(950, "results", 1, E, d, F, T, 0.0, E, E)
    r = make_runner(wl, threads=4)
    r.ctx.set_fusion(fused)
    r.ctx.set_top_k(k)
    ids = np.repeat(np.arange(E, dtype=np.int32), counts)[:T]
    np.random.default_rng(5).shuffle(ids)
    x, alpha = gen_x(wl, 0, T // k), gen_gate(wl, 0, T)
    xd, idd, ad, _ = r.to_device(x, ids, alpha)
    margin, n = 4096, T // k * d
    flat = torch.full((n + 2 * margin,), 0x7fc1, dtype=torch.uint16, device=r.dev)
    xs = torch.empty(n + 8, dtype=torch.uint16, device=r.dev)
    xs[shift:shift + n] = xd.view(torch.uint16).reshape(-1)
    x_at = xs[shift:shift + n].view(torch.bfloat16).view(T // k, d)
    lo = margin + shift
    y = flat[lo:lo + n].view(torch.bfloat16).view(T // k, d)
    for _ in range(2):
        flat.fill_(0x7fc1)                                  # the second pass writes every row again
        torch.cuda.synchronize()
        r.run(r.plan_all([ids]), [x_at], [idd], [ad], [y])
        r.sync()
    if k == 1:
        want = oracle_layer(wl, r, 0, x, ids, alpha)
    else:
        import oracle
        want = oracle.moe_forward_topk(x, ids.reshape(-1, k), alpha.reshape(-1, k), list(r.host_weights.numpy()), d, F)
    assert_close(bf16_tensor_to_f32(y), want, f"shift {shift}")
    outside = torch.cat([flat[:lo], flat[lo + n:]]).cpu().numpy()
    assert (outside == 0x7fc1).all()
    r.close()
