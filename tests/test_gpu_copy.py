"""The copy kernel: which experts it brings and where their bytes land, from one expert of eight tiles
(fewer than the grid has wavefronts) to waves of several, on copy streams of every width."""
import numpy as np
import pytest
import torch

from gpu_util import say
from paper_2310_18859_amd.runner import MoERunner
from test_gpu_layer import slot_order

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("copy_cus", [0, 8, 16, 24])
@pytest.mark.parametrize("d,F,experts", [(128, 128, [4]), (128, 384, [0, 2, 5]), (640, 256, [1, 2, 3, 4]),
                                         (768, 3072, [0, 1, 2, 3, 5])])
def test_slots_hold_the_experts(d, F, experts, copy_cus):
    say(f"copy kernel: d={d} F={F} experts={experts} copy_cus={copy_cus}")
    E = 6
    r = MoERunner(1, E, d, F, E, E, 64, copy_cus=copy_cus)
    r.alloc_host_weights()[:] = np.random.default_rng(d + F).integers(0, 1 << 16, (E, 2 * d * F), dtype=np.uint16)
    before = r.host_weights.numpy().copy()
    r.pool.fill_(0xA5)
    torch.cuda.synchronize()
    plan = r.ctx.moe_plan(0, np.array(experts, dtype=np.int32))
    r.ctx.expert_prefetch(plan, 0, r.copy)
    r.copy.synchronize()
    pool = r.pool.view(torch.uint16).reshape(E, -1).cpu().numpy()
    used = {plan.slot[e]: e for e in experts}
    for s in range(E):
        want = slot_order(before[used[s]], d, F) if s in used else np.full(2 * d * F, 0xA5A5, np.uint16)
        assert np.array_equal(pool[s], want), f"slot {s}"
    assert np.array_equal(r.host_weights.numpy(), before)
    r.close()
