"""Alg. 1 on a grid of tiles: the device's checks of a batch's lists, capture, and the walk against the oracle."""
import numpy as np
import pytest

import oracle
import ptycho_synth as ps
import paper_2205_06327_amd as pt
from paper_2205_06327_amd import _binding as B
from paper_2205_06327_amd.tilewalk import Alg1Walk, TileWalk

from gpu_helpers import context, problem, rel_l2, say, to_dev

pytestmark = pytest.mark.gpu


def _tiles(spec, plan, obj):
    """(V, AccBuf, gradient) of every tile, each in memory of its own."""
    import torch
    out = []
    for p in plan.plans:
        ey0, ex0, eh, ew = p.box
        V = obj[:, ey0:ey0 + eh, ex0:ex0 + ew].clone(memory_format=torch.contiguous_format)
        out.append((p.tile, p.box, V, torch.zeros_like(V), torch.zeros_like(V)))
    return out


@pytest.mark.parametrize("S", [1, 3])
def test_batch_step_checks_its_lists(S):
    """Jobs whose index is no position, and positions listed under another tile than their own, are
    skipped and reported; the others take their step as without them, and every gradient buffer is zero
    again.  Segments on the device that reach beyond the batch are cut to it."""
    import torch
    spec = ps.with_overrides(ps.workload("2d-256-m64"), S=S, W=192, ny=13, nx=13, step=8, tiles=(2, 2), halo=48)
    say(f"batch step lists, S={S}")
    d = ps.build_inputs(spec)
    plan = TileWalk(d["pos"], spec.W, spec.W, spec.M, spec.tiles, spec.halo)
    dev = "cuda:0"
    obj = torch.tensor(d["obj_eval"], dtype=torch.complex64, device=dev)
    probe = torch.tensor(d["probe"], dtype=torch.complex64, device=dev)
    pos = torch.tensor(plan.pos_sorted, device=dev)
    g = torch.Generator(device=dev)
    g.manual_seed(4)
    meas = torch.rand((plan.n, spec.M, spec.M), generator=g, device=dev) * 50
    owner = np.concatenate([np.full(p.hi - p.lo, k) for k, p in enumerate(plan.plans)]).astype(np.int32)
    tile_of_pos = torch.tensor(owner, device=dev)
    ctx = context(spec, plan.n + 8)
    step = 1e-7

    def run(lists, device_segments=None):
        tiles = _tiles(spec, plan, obj)
        seg = np.concatenate([[0], np.cumsum([len(x) for x in lists])]).astype(np.int32)
        index = torch.tensor(np.concatenate(lists), dtype=torch.int32, device=dev)
        dseg = torch.tensor(seg if device_segments is None else device_segments(seg), dtype=torch.int32, device=dev)
        losses = torch.full((len(tiles),), -1.0, dtype=torch.float64, device=dev)
        B.ptycho_tiles_batch_step(ctx, B.tile_states(ctx, tiles), tile_of_pos, probe, pos, meas, index, dseg, seg,
                                  step, losses)
        try:
            ctx.check()
            status = None
        except pt.PtychoError as e:
            status = e.name
        for _, _, V, acc, grad in tiles:
            assert not bool(torch.view_as_real(grad).any())
        return status, tiles, losses.cpu().numpy()

    def same(a, b):
        np.testing.assert_allclose(a[2], b[2], rtol=1e-12)
        for (_, _, V, acc, _), (_, _, W, bcc, _) in zip(a[1], b[1]):
            assert rel_l2(acc.cpu().numpy(), bcc.cpu().numpy()) <= 1e-6  # the order of the atomics
            assert rel_l2(V.cpu().numpy(), W.cpu().numpy()) <= 1e-6

    lists = [list(range(p.lo, p.lo + 9)) for p in plan.plans]
    good = run(lists)
    assert good[0] is None and float(good[2].min()) > 0
    assert all(bool(acc.abs().max() > 0) for _, _, _, acc, _ in good[1])
    for bad in (-1, plan.n, 2 ** 31 - 1, -2 ** 31):
        for k in (0, 2, 3):
            got = run([x[:4] + [bad] + x[4:] if j == k else x for j, x in enumerate(lists)])
            assert got[0] == "PTYCHO_E_BOUNDS"
            same(got, good)
    other = plan.plans[3].lo + 20  # owned by tile 3, listed under tile 1
    got = run([x + [other] if k == 1 else x for k, x in enumerate(lists)])
    assert got[0] == "PTYCHO_E_ASSIGN"
    same(got, good)
    got = run(lists, lambda seg: np.where(np.arange(5) == 4, seg[4] + 1000, np.where(np.arange(5) == 0, -7, seg)))
    assert got[0] is None
    same(got, good)
    # the device's segments put tile 0's last job under tile 1: skipped
    got = run(lists, lambda seg: seg - (np.arange(5) == 1))
    assert got[0] == "PTYCHO_E_ASSIGN"
    same(got, run([lists[0][:-1]] + lists[1:]))


def test_captured_iteration_replays_beside_other_calls():
    """The first iteration of a walk goes into a graph; between the replays another walk and an all-tiles
    gradient use the same context.  Every replay is an iteration of the walk, as in eager mode."""
    import torch
    from paper_2205_06327_amd.tilewalk import AllTilesWalk
    spec = ps.with_overrides(ps.workload("2d-256-m64"), S=2, W=192, ny=13, nx=13, step=8, tiles=(2, 2), halo=48)
    say("captured Alg. 1 iteration")
    d = ps.build_inputs(spec)
    dev = "cuda:0"
    obj = torch.tensor(d["obj_eval"], dtype=torch.complex64, device=dev)
    probe = torch.tensor(d["probe"], dtype=torch.complex64, device=dev)
    plan = TileWalk(d["pos"], spec.W, spec.W, spec.M, spec.tiles, spec.halo)
    half = TileWalk(d["pos"][::2], spec.W, spec.W, spec.M, spec.tiles, spec.halo)
    g = torch.Generator(device=dev)
    g.manual_seed(8)
    meas = torch.rand((plan.n, spec.M, spec.M), generator=g, device=dev) * 50
    ctx = context(spec, plan.n)
    pt.ptycho_forward(ctx, obj, probe, torch.tensor(plan.pos_sorted, device=dev))
    eager, walk = (Alg1Walk(ctx, plan, obj.clone(), probe, meas, 1e-7, 16, 2) for _ in range(2))
    other = Alg1Walk(ctx, half, obj.clone(), probe, meas[:half.n], 1e-7, 8, 1)
    tiles = AllTilesWalk(ctx, plan)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        loss = walk.iteration()
    grad, V, W = (torch.empty_like(obj) for _ in range(3))
    for _ in range(3):
        other.iteration()
        tiles.step(obj, probe, meas, grad)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        want = float(eager.iteration().item())
        assert float(loss.item()) == pytest.approx(want, rel=1e-6)
        walk.stitch(V)
        eager.stitch(W)
        assert rel_l2(V.cpu().numpy(), W.cpu().numpy()) <= 1e-6
    assert rel_l2(V.cpu().numpy(), obj.cpu().numpy()) > 1e-5  # it moved
    assert ctx.check() == 0


def _walk(spec, d, batch, T, extra=0):
    import torch
    t = to_dev(d)
    plan = TileWalk(d["pos"], spec.W, spec.W, spec.M, spec.tiles, spec.halo)
    meas = t["meas"][torch.tensor(plan.order, device="cuda:0")]
    meas = torch.cat([meas, meas[:extra]])
    alpha = 0.5 * oracle.gd_step_size(d["probe"], d["pos"], spec.W, spec.W, spec.S)
    return t, alpha, Alg1Walk(context(spec, spec.n), plan, t["obj"], t["probe"], meas, alpha, batch, T)


def _matches_oracle(spec, d, t, alpha, walk, batch, T, iterations=2):
    import torch
    losses = []
    for _ in range(iterations):
        losses.append(float(walk.iteration().item()))
        assert not any(bool(torch.view_as_real(g).any()) for g in walk.gbuf)  # zero between calls
    assert walk.check() == 0
    V = torch.empty_like(t["obj"])
    walk.stitch(V)
    ref_l, ref_V = oracle.alg1_tiles(d["obj_eval"], d["probe"], d["pos"], d["meas"], d["H"], spec.tiles, spec.halo,
                                     alpha, batch, T, iterations)
    np.testing.assert_allclose(losses, ref_l, rtol=1e-4)
    # every FP32 write of V_k rounds by up to 2^-24 |V|, |V| ~ 1, against the size of the update
    V0 = d["obj_eval"].astype(np.complex128)
    dV = ref_V - V0
    writes = iterations * (walk.steps + -(-walk.steps // T))
    tol = 1e-4 + writes * 2.0 ** -24 * np.linalg.norm(V0) / np.linalg.norm(dV)
    assert rel_l2(V.cpu().numpy() - V0, dV) <= tol


@pytest.mark.parametrize("tiles,S", [((3, 1), 1), ((1, 1), 1), ((1, 1), 2), ((3, 1), 2)])
def test_tiles_keep_their_own_copies(tiles, S):
    """Tiles of full-width rows: the boxes of a single slice are views of the object that need no copy to be
    contiguous, and neighbouring ones overlap.  Every V_k is a copy, and the object is not written."""
    import torch
    spec = ps.with_overrides(ps.workload("2d-256-m64"), W=192, S=S, ny=13, nx=13, step=8, tiles=tiles, halo=32)
    say(f"Alg. 1, tiles {tiles}, S={S}")
    d = problem(spec)
    t, alpha, walk = _walk(spec, d, 8, 2)
    before = t["obj"].clone()
    _matches_oracle(spec, d, t, alpha, walk, 8, 2)
    assert torch.equal(t["obj"], before)


def test_more_patterns_than_positions():
    """Patterns beyond the plan's positions are not looked at."""
    spec = ps.with_overrides(ps.workload("2d-256-m64"), W=192, S=2, ny=9, nx=9, step=8, tiles=(2, 2), halo=48)
    say("Alg. 1 with more patterns than positions")
    d = problem(spec)
    t, alpha, walk = _walk(spec, d, 8, 2, extra=3)
    _matches_oracle(spec, d, t, alpha, walk, 8, 2)


def _scattered(M, S, H_W, n, tiles, halo, seed, within=None):
    """n positions at random (window centres below `within` of the object's width only, when given)."""
    spec = ps.with_overrides(ps.workload("2d-256-m64" if M == 64 else "ms8-1024-m128"), W=H_W, S=S, ny=2, nx=2, step=4,
                             tiles=tiles, halo=halo, noise=False)
    d = ps.build_inputs(spec)
    d["H"] = oracle.fresnel_propagator(spec.M, spec.wavelength_A, spec.dz_A, spec.pixel_A)
    rng = np.random.default_rng(seed)
    top = H_W - M
    pos = np.stack([rng.integers(0, top + 1, n), rng.integers(0, (top if within is None else within) + 1, n)], 1)
    d["pos"] = np.ascontiguousarray(pos, dtype=np.int32)
    d["meas"] = oracle.forward(d["obj_true"], d["probe"], d["pos"], d["H"]).astype(np.float32)
    return spec, d


@pytest.mark.parametrize("M,S,W,n,tiles,halo,batch,T,within", [
    (128, 2, 301, 420, (2, 2), 64, 150, 1, None),  # odd boxes (atomics staged), more jobs than workgroups
    (128, 3, 304, 300, (2, 1), 64, 200, 2, None),  # boxes of a whole number of lines, rolled
    (64, 1, 190, 2500, (2, 2), 33, 900, 1, None),  # register sums across tiles, runs of several jobs
    (64, 1, 192, 900, (2, 3), 32, 1, 40, None),    # a position at a time
    (64, 2, 600, 150, (1, 2), 40, 20, 3, 200),     # rows wider than a step of the update; a tile without positions
])
def test_walk_over_launch_shapes(M, S, W, n, tiles, halo, batch, T, within):
    """Batches that give a workgroup several jobs, of several tiles with boxes of their own width; odd and
    whole-line boxes, one and more slices, tiles without positions and batches of uneven size."""
    import torch
    say(f"Alg. 1, M={M} S={S} W={W} n={n} tiles {tiles} batch {batch}")
    spec, d = _scattered(M, S, W, n, tiles, halo, 17, within)
    t = to_dev(d)
    plan = TileWalk(d["pos"], W, W, M, tiles, halo)
    alpha = 0.5 * oracle.gd_step_size(d["probe"], d["pos"], W, W, S)
    meas = t["meas"][torch.tensor(plan.order, device="cuda:0")]
    walk = Alg1Walk(context(spec, n), plan, t["obj"], t["probe"], meas, alpha, batch, T)
    if within is not None:
        assert min(p.hi - p.lo for p in plan.plans) == 0
    _matches_oracle(spec, d, t, alpha, walk, batch, T)
