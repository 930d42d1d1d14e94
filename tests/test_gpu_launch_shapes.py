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
