"""Single-slice gradients of 64-windows, which are summed in registers along a workgroup's run of positions."""
import numpy as np
import pytest

import ptycho_synth as ps
import paper_2205_06327_amd as pt
from paper_2205_06327_amd.tilewalk import TileWalk

from gpu_helpers import context, rel_l2, say

pytestmark = pytest.mark.gpu


def test_tiles_sharing_a_gradient_buffer():
    """Two tiles with boxes of one shape may be given the same buffer: it receives the sum of both, although
    the same object column lies at another place of it for each tile.  Runs cross from one tile to the other
    within a scan row."""
    import torch
    say("two tiles share a gradient buffer")
    spec = ps.with_overrides(ps.workload("2d-256-m64"), S=1, W=256, ny=2, nx=2, step=4, noise=False)
    d = ps.build_inputs(spec)
    H, W, halo = 256, 256, 32
    pos = np.array([(y, x) for y in range(0, 111, 3) for x in range(0, W - 63, 3)], dtype=np.int32)
    plan = TileWalk(pos, H, W, 64, (1, 4), halo)
    obj = torch.tensor(d["obj_eval"], dtype=torch.complex64, device="cuda:0")
    probe = torch.tensor(d["probe"], dtype=torch.complex64, device="cuda:0")
    dev_pos = torch.tensor(pos, device="cuda:0")
    owner = torch.tensor(pt.bin_positions(pos, H, W, 64, 1, 4), device="cuda:0")
    g = torch.Generator(device="cuda:0")
    g.manual_seed(6)
    meas = torch.rand((len(pos), 64, 64), generator=g, device="cuda:0") * 50
    ctx = context(spec, len(pos))
    bufs = [torch.empty((1, p.box[2], p.box[3]), dtype=torch.complex64, device="cuda:0") for p in plan.plans]
    assert bufs[1].shape == bufs[2].shape

    def grads(b):
        pt.ptycho_tiles_grad(ctx, obj, [(p.tile, p.box, b[k]) for k, p in enumerate(plan.plans)], halo, owner, probe,
                             dev_pos, meas)
        assert ctx.check() == 0
        return [x.cpu().numpy() for x in b]
    one = grads(bufs)
    shared = [torch.empty_like(b) for b in bufs]
    shared[2] = shared[1]
    got = grads(shared)
    for k in (0, 3):
        assert rel_l2(got[k], one[k]) <= 1e-6
    assert rel_l2(got[1], one[1] + one[2]) <= 1e-6
