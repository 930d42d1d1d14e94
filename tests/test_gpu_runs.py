"""Runs of consecutive positions per workgroup: whole rounds of runs with a remainder, and register sums
along runs that hold rejected positions, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
import ptycho_synth as ps
import paper_2205_06327_amd as pt

from gpu_helpers import context, rel_l2, say, to_dev

pytestmark = pytest.mark.gpu

TOL_G, TOL_L = 1e-4, 1e-5  # FP32 kernels against the FP64 oracle, as in the parity tests


def _scan(M, S, n, W, step):
    """A raster of n positions, again from the top where it is full, with the patterns of 40 of them in turn."""
    spec = ps.with_overrides(ps.workload("2d-256-m64" if M == 64 else "2d-1024-m128"), S=S, W=W, ny=2, nx=2, step=step,
                             noise=False)
    d = ps.build_inputs(spec)
    d["H"] = oracle.fresnel_propagator(spec.M, spec.wavelength_A, spec.dz_A, spec.pixel_A)
    xy = np.arange(0, W - M + 1, step)
    raster = np.array([(y, x) for y in xy for x in xy], dtype=np.int32)
    d["pos"] = np.ascontiguousarray(raster[np.arange(n) % len(raster)])
    some = raster[:: max(1, len(raster) // 40)]
    I = oracle.forward(d["obj_true"], d["probe"], some, d["H"]).astype(np.float32)
    d["meas"] = I[np.arange(n) % len(some)]
    return spec, d


def _runs(n, grid, run):
    """The positions of every workgroup, in order: 8 contiguous chunks, one per XCD; rounds of runs, then the
    rest of a chunk split evenly."""
    out = []
    for b in range(grid):
        x, k = b % 8, b // 8
        gx = (grid - x + 7) // 8
        lo, hi = x * n // 8, (x + 1) * n // 8
        rounds = (hi - lo) // (gx * run)
        p = [lo + (j * gx + k) * run + i for j in range(rounds) for i in range(run)]
        r0 = lo + rounds * gx * run
        base, more = divmod(hi - r0, gx)
        first = r0 + k * base + min(k, more)
        out.append(p + list(range(first, first + base + (k < more))))
    assert sorted(sum(out, [])) == list(range(n))
    return out


@pytest.mark.parametrize("M,n", [(64, 6144), (64, 6149), (64, 6920), (128, 2048), (128, 2085)])
def test_whole_rounds_of_runs(M, n):
    """Two-slice gradients take runs of 8; 768 workgroups of 64-windows or 256 of 128-windows fill a round with
    6144 or 2048 positions.  Every position is taken once, at its place."""
    import torch
    say(f"rounds of runs M={M} n={n}")
    spec, d = _scan(M, 2, n, M + 40, 5)
    t = to_dev(d)
    ctx = context(spec, n)
    per = torch.full((n,), -1.0, dtype=torch.float64, device="cuda:0")
    loss, G = pt.ptycho_loss_grad(ctx, t["obj"], t["probe"], t["pos"], t["meas"], loss_per_pos=per)
    assert ctx.check() == 0
    period = np.lcm(len(np.unique(d["pos"], axis=0)), len(np.unique(d["meas"].reshape(n, -1), axis=0)))
    m = int(min(n, period))  # positions and patterns repeat: the oracle takes one period, weighted
    L_all, f, G_all = oracle.loss_and_gradient(d["obj_eval"], d["probe"], d["pos"][:m], d["meas"][:m], d["H"])
    whole, rest = divmod(n, m)
    L_ref, G_ref = whole * L_all, whole * G_all
    if rest:
        L_rest, _, G_rest = oracle.loss_and_gradient(d["obj_eval"], d["probe"], d["pos"][:rest], d["meas"][:rest], d["H"])
        L_ref, G_ref = L_ref + L_rest, G_ref + G_rest
    np.testing.assert_allclose(per.cpu().numpy(), f[np.arange(n) % m], rtol=1e-4)
    assert abs(float(loss.item()) - L_ref) <= TOL_L * L_ref
    assert rel_l2(G.cpu().numpy(), G_ref) <= TOL_G


@pytest.mark.parametrize("where", ["first", "middle", "last", "many"])
def test_rejected_positions_within_a_run(where):
    """Single-slice gradients of 64-windows are held in registers along a run (6 or 7 positions here).  A
    rejected position at its start, while values are held, at its end, or several of them leave the rest whole."""
    n = 5000
    say(f"rejected positions, {where} in a run")
    spec, d = _scan(64, 1, n, 64 + 45, 3)
    rng = np.random.default_rng(11)
    bad = []
    for p in [r for r in _runs(n, 768, 1 << 20) if rng.random() < 0.2]:
        assert len(p) in (6, 7)
        bad += {"first": p[:1], "middle": p[2:4], "last": p[-1:], "many": p[1:5:2] + p[-1:]}[where]
    bad = np.array(bad)
    keep = np.setdiff1d(np.arange(n), bad)
    pos = d["pos"].copy()
    pos[bad[::2]] = (46, 3)  # a row below the object
    pos[bad[1::2]] = (3, -1)
    t = to_dev(dict(d, pos=pos))
    ctx = context(spec, n)
    loss, G = pt.ptycho_loss_grad(ctx, t["obj"], t["probe"], t["pos"], t["meas"])
    with pytest.raises(pt.PtychoError) as e:
        ctx.check()
    assert e.value.name == "PTYCHO_E_BOUNDS"
    L_ref, _, G_ref = oracle.loss_and_gradient(d["obj_eval"], d["probe"], d["pos"][keep], d["meas"][keep], d["H"])
    assert abs(float(loss.item()) - L_ref) <= TOL_L * L_ref
    assert rel_l2(G.cpu().numpy(), G_ref) <= TOL_G
