"""Consecutive layers of equally many tokens are sorted by one launch, all but the last of them into the
x_perm region: groups of more layers than one launch takes, layers of other sizes between them, regions that
hold no second sort, and ids at an odd address.  Against the same layers one call at a time, bit for bit, and
against the oracle."""
import numpy as np
import pytest
import torch

from gpu_util import assert_close, bf16_tensor_to_f32, make_runner, oracle_layer, say
from workloads import Workload, gen_gate, gen_ids, gen_x

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,E,d,F,sizes,odd", [
    ("more-than-a-launch", 16, 128, 256, [700] * 17, ()),           # groups of 8, 8 and 1
    ("sizes-change", 16, 128, 256, [300, 300, 64, 301, 301, 300, 2100, 2100], ()),
    ("one-round-a-wavefront", 16, 128, 256, [511, 512, 512, 513, 513], ()),
    ("no-room", 200, 128, 128, [8] * 3, ()),                        # x_perm is smaller than one layer's sort
    ("room-for-few", 200, 128, 128, [64] * 7, ()),                  # ... holds fewer than a launch sorts
    ("chunks", 8, 128, 256, [4097, 4097, 5000, 5000, 5000], ()),
    ("chunks-odd-address", 8, 128, 256, [5000] * 4, (1, 3)),        # ids are not on a 16-byte boundary
    ("chunks-odd-first-and-last", 8, 128, 256, [4100] * 9, (0, 7, 8)),
    ("chunks-all-odd", 8, 128, 256, [4100] * 3, (0, 1, 2)),
    ("one-workgroup-odd-address", 8, 128, 256, [999] * 3, (0,)),
])
def test_layers_sorted_together(name, E, d, F, sizes, odd):
    say(f"sort groups: {name} E={E} sizes={sizes}")
    L = len(sizes)
    wl = Workload(660 + L, name, L, E, d, F, max(sizes), 1.0, L * E, E)
    r = make_runner(wl)
    ins = [(gen_x(wl, l)[:t], gen_ids(wl, l)[:t], gen_gate(wl, l)[:t]) for l, t in enumerate(sizes)]
    dev = [r.to_device(*i) for i in ins]
    ids = []
    for l, t in enumerate(sizes):
        pad = 1 if l in odd else 0
        buf = torch.empty(t + pad, dtype=torch.int32, device=r.dev)
        buf[pad:].copy_(dev[l][1])
        ids.append(buf[pad:])
        assert (ids[l].data_ptr() % 16 == 4 * pad)
    alone = []
    for l in range(L):
        x, i, a, y = dev[l]
        plan = r.ctx.moe_plan(l, ins[l][1])
        torch.cuda.synchronize()
        r.ctx.moe_layer_forward(plan, x, i, a, y, r.workspace, r.compute, r.copy)
        r.sync()
        alone.append(y.clone())
        assert_close(bf16_tensor_to_f32(y), oracle_layer(wl, r, l, *ins[l]), f"{name} layer {l}")
        y.fill_(7.0)                                                 # every row must be overwritten
    torch.cuda.synchronize()
    r.run(r.plan_all([i[1] for i in ins]), [v[0] for v in dev], ids, [v[2] for v in dev], [v[3] for v in dev])
    r.sync()
    for l in range(L):
        assert torch.equal(dev[l][3].view(torch.uint16), alone[l].view(torch.uint16)), f"{name} layer {l}"
    r.close()
