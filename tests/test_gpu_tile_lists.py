"""Whole-grid calls between tile buffers (one launch for a list of boxes) against the box-by-box calls on
the GPU, bit for bit: both add the same terms in the same order.  Views that are not dense take the
box-by-box route."""
import numpy as np
import pytest

import paper_2205_06327_amd as pt
from paper_2205_06327_amd import _binding as B
from paper_2205_06327_amd.tilewalk import TileWalk, directional_passes, neighbour_add, stitch_interiors

from gpu_helpers import say

pytestmark = pytest.mark.gpu


def _setup(S, H, W, tiles, halo):
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(7)
    plan = TileWalk(np.zeros((1, 2), np.int32), H, W, 64, tiles, halo)
    dense = [torch.randn((S, p.box[2], p.box[3]), dtype=torch.complex64, generator=g, device="cuda:0")
             for p in plan.plans]

    def views():  # the same values behind a longer row pitch
        out = []
        for b in dense:
            v = torch.zeros((b.shape[0], b.shape[1], b.shape[2] + 3), dtype=torch.complex64, device="cuda:0")[:, :, 1:-2]
            v.copy_(b)
            out.append(v)
        return out
    return pt.Context(64, S, 0.0197, 2.0, 0.1, 16), plan, dense, views


# one tile; a row and a column of tiles; odd sizes; more tiles than one list holds (25 tiles with 9 sources
# each); tiles smaller than the halo, where boxes of tiles two and three apart overlap
@pytest.mark.parametrize("S,H,W,tiles,halo", [(1, 70, 67, (1, 1), 8), (3, 65, 500, (1, 4), 33), (2, 301, 77, (3, 1), 20),
                                              (2, 333, 517, (3, 4), 31), (1, 320, 330, (5, 5), 32),
                                              (1, 200, 180, (6, 7), 64)])
def test_grid_calls_equal_box_calls(S, H, W, tiles, halo):
    import torch
    say(f"tile lists S={S} {H}x{W} tiles {tiles} halo {halo}")
    ctx, plan, dense, views = _setup(S, H, W, tiles, halo)
    # stitch: the sum of all boxes, and the interiors
    ref = torch.empty((S, H, W), dtype=torch.complex64, device="cuda:0")
    B.ptycho_zero_gradient(ctx, ref)
    for p, b in zip(plan.plans, dense):
        B.ptycho_tile_accumulate(ctx, b, p.box, ref)
    wide = torch.full((S, H, W + 5), 9.0, dtype=torch.complex64, device="cuda:0")
    got = wide[:, :, 2:-3]
    B.ptycho_tiles_stitch(ctx, [(p.tile, p.box, b) for p, b in zip(plan.plans, dense)], got)
    assert torch.equal(got, ref)
    assert bool((wide[:, :, :2] == 9).all()) and bool((wide[:, :, -3:] == 9).all())
    inner, inner_ref = torch.empty_like(ref), torch.empty_like(ref)
    stitch_interiors(ctx, plan, dense, inner)
    stitch_interiors(ctx, plan, views(), inner_ref)
    assert torch.equal(inner, inner_ref)
    # neighbour addition
    acc, acc_ref = [torch.empty_like(b) for b in dense], views()
    neighbour_add(ctx, plan, dense, acc)
    neighbour_add(ctx, plan, views(), acc_ref)
    for a, r in zip(acc, acc_ref):
        assert torch.equal(a, r)
    # directional passes, in place
    a, r = [b.clone() for b in dense], views()
    directional_passes(ctx, plan, a)
    directional_passes(ctx, plan, r)
    for x, y in zip(a, r):
        assert torch.equal(x, y)


def test_grid_calls_refuse_bad_tables():
    import torch
    say("whole-grid calls refuse bad tables on the host")
    ctx, plan, dense, views = _setup(1, 200, 180, (2, 2), 16)
    out = torch.zeros((1, 200, 180), dtype=torch.complex64, device="cuda:0")
    tiles = [(p.tile, p.box, b) for p, b in zip(plan.plans, dense)]

    def code(call):
        with pytest.raises(pt.PtychoError) as e:
            call()
        return e.value.name
    assert code(lambda: B.ptycho_tiles_stitch(ctx, tiles[:3], out)) == "PTYCHO_E_SHAPE"  # not covered
    assert code(lambda: B.ptycho_tiles_stitch(ctx, tiles[:3] + tiles[:1], out)) == "PTYCHO_E_SHAPE"
    assert code(lambda: B.ptycho_tiles_stitch(ctx, tiles, out[:, :-1])) == "PTYCHO_E_SHAPE"  # box outside
    assert code(lambda: B.ptycho_tiles_stitch(ctx, tiles, out, 2)) == "PTYCHO_E_ARG"
    assert code(lambda: B.ptycho_tiles_neighbour_add(ctx, tiles, dense, (2, 2))) == "PTYCHO_E_ARG"  # shared memory
    assert code(lambda: B.ptycho_tiles_passes(ctx, tiles[:1] * 4, (2, 2))) == "PTYCHO_E_ARG"
    with pytest.raises(ValueError):
        B.ptycho_tiles_stitch(ctx, [(t, b, v) for (t, b, _), v in zip(tiles, views())], out)  # not dense
    assert float(out.abs().max()) == 0.0


def test_single_slice_tiles_of_64_windows():
    """Single-slice 64-windows are summed in registers along a workgroup's run of positions; in the
    all-tiles launch a run crosses from one tile's buffer to the next.  Against the undecomposed
    gradient, also into a gradient array larger than the tiled object (zero beyond it)."""
    import torch
    import ptycho_synth as ps
    from paper_2205_06327_amd.tilewalk import AllTilesWalk
    from gpu_helpers import context, rel_l2
    say("single-slice all-tiles launch, M=64")
    spec = ps.with_overrides(ps.workload("2d-256-m64"), W=256, ny=49, nx=49, step=4)
    d = ps.build_inputs(spec)
    obj = torch.tensor(d["obj_eval"], dtype=torch.complex64, device="cuda:0")
    probe = torch.tensor(d["probe"], dtype=torch.complex64, device="cuda:0")
    plan = TileWalk(d["pos"], spec.W, spec.W, spec.M, (3, 2), 32)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(2)
    meas = torch.rand((spec.n, spec.M, spec.M), generator=g, device="cuda:0") * 50
    ctx = context(spec, spec.n)
    ref_loss, ref = pt.ptycho_loss_grad(ctx, obj, probe, torch.tensor(plan.pos_sorted, device="cuda:0"), meas)
    walk = AllTilesWalk(ctx, plan)
    grad = torch.empty_like(obj)
    loss = float(walk.step(obj, probe, meas, grad).item())
    wide = torch.full((1, spec.W + 3, spec.W + 8), 5.0, dtype=torch.complex64, device="cuda:0")
    walk.step(obj, probe, meas, wide)
    assert walk.check() == 0
    assert abs(loss - float(ref_loss.item())) <= 1e-9 * loss
    assert rel_l2(grad.cpu().numpy(), ref.cpu().numpy()) <= 1e-6
    assert rel_l2(wide[:, :spec.W, :spec.W].cpu().numpy(), ref.cpu().numpy()) <= 1e-6
    assert float(wide[:, spec.W:].abs().max()) == 0.0 and float(wide[:, :, spec.W:].abs().max()) == 0.0
