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
