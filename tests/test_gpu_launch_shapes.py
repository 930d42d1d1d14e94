"""GPU parity at the edges of the launch shapes: position counts around the
workgroup and reduction widths, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import ptycho_synth as ps

from gpu_helpers import context, problem, rel_l2, say, to_dev

pytestmark = pytest.mark.gpu

TOL_G, TOL_L = 1e-4, 1e-5  # FP32 kernels against the FP64 oracle, as in the parity tests


@pytest.mark.parametrize("M,nx,ny", [(64, 1, 1), (64, 5, 13), (64, 32, 27), (128, 17, 1), (128, 13, 5), (128, 17, 16)])
def test_probe_gradient_partial_sums(M, nx, ny):
    """The partial sums of 1, 17, 65, 272 and 864 positions: fewer than, as many as and more than the 16
    waves and 4 loads of the reduction, and more positions than workgroups in flight (256 for
    128-windows, 768 for 64-windows)."""
    import torch
    import paper_2205_06327_amd as pt
    step = 4
    spec = ps.with_overrides(ps.workload("2d-256-m64" if M == 64 else "2d-1024-m128"), S=1, ny=ny, nx=nx, step=step,
                             W=M + step * (max(nx, ny) - 1) + 3, noise=True)
    say(f"probe gradient M={M} n={spec.n}")
    d = problem(spec)
    t = to_dev(d)
    ctx = context(spec, spec.n)
    pg = torch.empty_like(t["probe"])
    loss, G = pt.ptycho_loss_grad(ctx, t["obj"], t["probe"], t["pos"], t["meas"], probe_grad=pg)
    assert ctx.check() == 0
    L_ref, _, G_ref = oracle.loss_and_gradient(d["obj_eval"], d["probe"], d["pos"], d["meas"], d["H"])
    P_ref = oracle.probe_gradient(d["obj_eval"], d["probe"], d["pos"], d["meas"], d["H"])
    assert abs(float(loss.item()) - L_ref) <= TOL_L * L_ref
    assert rel_l2(G.cpu().numpy(), G_ref) <= TOL_G
    assert rel_l2(pg.cpu().numpy(), P_ref) <= TOL_G


@pytest.mark.parametrize("M", [64, 128])
@pytest.mark.parametrize("S", [1, 3])
@pytest.mark.parametrize("W_extra,view", [(32, 0), (32, 3), (25, 0)])
def test_window_offsets_from_a_line(M, S, W_extra, view):
    """Windows starting at every offset from a 128-byte line: a row pitch that is a multiple of 16
    (the windows are rolled to line alignment), the same as a view at column 3, and an odd pitch
    (no common alignment).  Intensities, loss, gradient and probe gradient."""
    import torch
    import paper_2205_06327_amd as pt
    W = M + W_extra
    spec = ps.with_overrides(ps.workload("2d-256-m64" if M == 64 else "ms8-1024-m128"), S=S, W=W, ny=2, nx=2, step=4,
                             noise=True)
    say(f"line offsets M={M} S={S} W={W} view={view}")
    d = problem(spec)
    d["pos"] = np.array([[(5 * k) % (W_extra + 1), k] for k in range(18)], dtype=np.int32)
    d["meas"] = ps.poisson_counts(oracle.forward(d["obj_true"], d["probe"], d["pos"], d["H"]), d["noise_seed"])
    t = to_dev(d)
    pitch = W if view == 0 else W + 16
    big = torch.zeros((S, W, pitch), dtype=torch.complex64, device="cuda:0")
    big[:, :, view:view + W] = t["obj"]
    obj = big[:, :, view:view + W]
    grad = torch.zeros_like(big)[:, :, view:view + W]
    ctx = context(spec, len(d["pos"]))
    I = pt.ptycho_forward(ctx, obj, t["probe"], t["pos"])
    pg = torch.empty_like(t["probe"])
    l2 = pt.ptycho_loss(ctx, obj, t["probe"], t["pos"], t["meas"])
    loss, _ = pt.ptycho_loss_grad(ctx, obj, t["probe"], t["pos"], t["meas"], grad=grad)
    G = grad.clone()
    pt.ptycho_loss_grad(ctx, obj, t["probe"], t["pos"], t["meas"], grad=grad, probe_grad=pg)
    assert ctx.check() == 0
    L_ref, _, G_ref = oracle.loss_and_gradient(d["obj_eval"], d["probe"], d["pos"], d["meas"], d["H"])
    P_ref = oracle.probe_gradient(d["obj_eval"], d["probe"], d["pos"], d["meas"], d["H"])
    assert rel_l2(I.cpu().numpy(), oracle.forward(d["obj_eval"], d["probe"], d["pos"], d["H"])) <= 1e-5
    for x in (loss, l2):
        assert abs(float(x.item()) - L_ref) <= TOL_L * L_ref
    assert rel_l2(G.cpu().numpy(), G_ref) <= TOL_G
    assert rel_l2(grad.cpu().numpy(), G_ref) <= TOL_G
    assert rel_l2(pg.cpu().numpy(), P_ref) <= TOL_G


@pytest.mark.parametrize("n", [9, 257, 775, 1541])
def test_runs_of_positions(n):
    """Every position is taken once whatever the count: fewer positions than workgroups, one more
    than a round, and whole rounds of runs with a remainder (768 workgroups of 64-windows)."""
    import paper_2205_06327_amd as pt
    nx = 41
    ny = -(-n // nx)
    spec = ps.with_overrides(ps.workload("2d-256-m64"), S=1, W=256, ny=ny, nx=nx, step=4, noise=True)
    say(f"runs of positions n={n}")
    d = problem(spec)
    d["pos"], d["meas"] = d["pos"][:n], d["meas"][:n]
    t = to_dev(d)
    ctx = context(spec, n)
    loss, G = pt.ptycho_loss_grad(ctx, t["obj"], t["probe"], t["pos"], t["meas"])
    assert ctx.check() == 0
    L_ref, _, G_ref = oracle.loss_and_gradient(d["obj_eval"], d["probe"], d["pos"], d["meas"], d["H"])
    assert abs(float(loss.item()) - L_ref) <= TOL_L * L_ref
    assert rel_l2(G.cpu().numpy(), G_ref) <= TOL_G


@pytest.mark.parametrize("M,n", [(64, 1700), (128, 600)])
@pytest.mark.parametrize("order", ["serpentine", "walk", "jumps"])
def test_single_slice_sums_over_a_run(M, n, order):
    """Single-slice gradients are summed in registers along a workgroup's run of positions: scan rows
    in both directions, a random walk with steps of 0 to 3 pixels in y and x (rows change within a
    run, positions repeat), and jumps beyond a window's width within a row; an odd row pitch, and a
    position outside the object in the middle of a run, which is skipped."""
    import torch
    import paper_2205_06327_amd as pt
    W = 2 * M + 61
    spec = ps.with_overrides(ps.workload("2d-256-m64" if M == 64 else "2d-1024-m128"), S=1, W=W, ny=2, nx=2, step=4,
                             noise=False)
    say(f"single-slice sums M={M} n={n} {order}")
    rng = np.random.default_rng(3)
    top = W - M
    if order == "serpentine":
        xs = np.arange(0, top + 1, 5)
        rows = [np.stack([np.full(len(xs), 3 * r % (top + 1)), xs if r % 2 == 0 else xs[::-1]], 1)
                for r in range(-(-n // len(xs)))]
        pos = np.concatenate(rows)[:n]
    elif order == "walk":
        d = rng.integers(-3, 4, size=(n, 2))
        d[rng.random(n) < 0.6, 0] = 0
        pos = np.abs(np.cumsum(d, 0) + top // 2) % (2 * top)
        pos = np.where(pos > top, 2 * top - pos, pos)
    else:
        pos = np.stack([np.repeat(rng.integers(0, top + 1, -(-n // 7)), 7)[:n], rng.integers(0, 2, n) * (M + 30)], 1)
    pos = np.ascontiguousarray(pos, dtype=np.int32)
    d = ps.build_inputs(spec)
    d["H"] = oracle.fresnel_propagator(spec.M, spec.wavelength_A, spec.dz_A, spec.pixel_A)
    some = rng.permutation(n)[:60]  # patterns of a few positions, repeated: the oracle's cost is in the gradient
    I = oracle.forward(d["obj_true"], d["probe"], pos[some], d["H"]).astype(np.float32)
    d["pos"], d["meas"] = pos, I[np.arange(n) % len(some)]
    t = to_dev(d)
    ctx = context(spec, n + 1)
    bad = n // 2
    dev_pos = torch.cat([t["pos"][:bad], torch.tensor([[top + 1, 0]], dtype=torch.int32, device="cuda:0"), t["pos"][bad:]])
    dev_meas = torch.cat([t["meas"][:bad], t["meas"][:1], t["meas"][bad:]])
    loss, G = pt.ptycho_loss_grad(ctx, t["obj"], t["probe"], dev_pos.contiguous(), dev_meas)
    with pytest.raises(pt.PtychoError) as e:
        ctx.check()
    assert e.value.name == "PTYCHO_E_BOUNDS"
    L_ref, _, G_ref = oracle.loss_and_gradient(d["obj_eval"], d["probe"], d["pos"], d["meas"], d["H"])
    assert abs(float(loss.item()) - L_ref) <= TOL_L * L_ref
    assert rel_l2(G.cpu().numpy(), G_ref) <= TOL_G
    # the same positions through the probe-gradient launch, which adds every window on its own
    pg = torch.empty_like(t["probe"])
    loss2, G2 = pt.ptycho_loss_grad(ctx, t["obj"], t["probe"], t["pos"], t["meas"], probe_grad=pg)
    assert ctx.check() == 0 and float(loss2.item()) == pytest.approx(float(loss.item()), rel=1e-12)
    assert rel_l2(G2.cpu().numpy(), G.cpu().numpy()) <= 1e-6


@pytest.mark.parametrize("M", [64, 128])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_intensities_into_any_float_address(M, offset):
    """Intensities are stored 16 bytes per lane; the output may start at any float."""
    import torch
    import paper_2205_06327_amd as pt
    spec = ps.with_overrides(ps.workload("2d-256-m64" if M == 64 else "ms8-1024-m128"), S=2, W=M + 20, ny=3, nx=3, step=7,
                             noise=False)
    say(f"intensities at float offset {offset}, M={M}")
    d = problem(spec)
    t = to_dev(d)
    n = spec.n
    buf = torch.full((offset + n * M * M + 5,), -1.0, device="cuda:0")
    out = buf[offset:offset + n * M * M].view(n, M, M)
    pt.ptycho_forward(context(spec, n), t["obj"], t["probe"], t["pos"], intens=out)
    assert rel_l2(out.cpu().numpy(), oracle.forward(d["obj_eval"], d["probe"], d["pos"], d["H"])) <= 1e-5
    assert bool((buf[:offset] == -1).all()) and bool((buf[offset + n * M * M:] == -1).all())


@pytest.mark.parametrize("n", [1, 7, 8, 9, 15, 100, 255])
def test_a_block_per_position(n):
    """Every pattern is written once when the launch has a workgroup per position, whatever the count
    is modulo the 8 XCDs, and again in the order of the positions."""
    import torch
    import paper_2205_06327_amd as pt
    spec = ps.with_overrides(ps.workload("2d-1024-m128"), S=1, W=160, ny=16, nx=16, step=2, noise=False)
    say(f"a block per position, n={n}")
    d = ps.build_inputs(spec)
    pos = np.ascontiguousarray(d["pos"][:n])
    H = oracle.fresnel_propagator(spec.M, spec.wavelength_A, spec.dz_A, spec.pixel_A)
    obj = torch.tensor(d["obj_eval"], dtype=torch.complex64, device="cuda:0")
    probe = torch.tensor(d["probe"], dtype=torch.complex64, device="cuda:0")
    out = torch.full((n, spec.M, spec.M), -1.0, device="cuda:0")
    ctx = context(spec, n)
    pt.ptycho_forward(ctx, obj, probe, torch.tensor(pos, device="cuda:0"), intens=out)
    assert ctx.check() == 0
    ref = oracle.forward(d["obj_eval"], d["probe"], pos, H)
    for i in range(n):
        assert rel_l2(out[i].cpu().numpy(), ref[i]) <= 1e-5, i
