"""Timed cases of the ptychography library: the calls a reconstruction program makes.

A case is one call pattern ("kind") with its sizes:

  forward    diffraction patterns of a scan (simulation; an acquisition preview asks for one pattern)
  grad       loss and object gradient of a whole scan (one step of a reconstruction)
  train      torch autograd: loss of a real potential, then backward (loss kernel + gradient kernel)
  probe      loss, object gradient and probe gradient (joint refinement)
  subpixel   real-valued scan positions: shifted probes, then loss and gradient with one probe each
  tiles      the decomposition with every tile's gradient in one launch, and the stitch
  batch      one gradient-descent iteration over many small uneven reconstructions (a graph replay)
  exchange   tile gradients added between neighbours, and the interiors stitched
  alg1       one iteration of the tiled reconstruction with delayed accumulation

Inputs are synthetic: jittered lattices of Gaussian atoms as phase slices, a defocused aperture
probe, a raster scan (optionally jittered by whole pixels, as a corrected stage reports it) and
Poisson counts of the patterns, evaluated at a nearby object.  They come from the seed through
torch alone, so two versions of the library see the same numbers.
"""
from __future__ import annotations

import math
import random

import torch

import paper_2205_06327_amd as pt
from paper_2205_06327_amd.autograd import amplitude_loss_potential
from paper_2205_06327_amd.batch import Batch, Recon
from paper_2205_06327_amd.tilewalk import AllTilesWalk, Alg1Walk, DecomposedTileWalk, TileWalk, stitch_interiors

WAVELENGTH, DZ, PIXEL = 0.0197, 2.0, 0.1  # 300 keV electrons, 2 Angstrom slices, 0.1 Angstrom pixels
PHYSICS = (WAVELENGTH, DZ, PIXEL)
DEV = "cuda:0"


def _case(name, kind, M, S, H, W, ny, nx, step, jitter=0, dose=1e5, strength=0.05, **more):
    c = {"kind": kind, "M": M, "S": S, "H": H, "W": W, "ny": ny, "nx": nx, "step": step, "jitter": jitter,
         "dose": dose, "strength": strength}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: one pattern of a small object (a preview while aligning); latency and launches
        _case("forward-one-m64", "forward", 64, 1, 256, 256, 1, 1, 8, strength=0.3),
        # simulating a whole single-slice scan
        _case("forward-2d-1024-m128", "forward", 128, 1, 1024, 1024, 64, 64, 14, strength=0.3),
        # one reconstruction step of a small single-slice scan: 256 positions, one per CU
        _case("grad-2d-256-m64", "grad", 64, 1, 256, 256, 16, 16, 8, strength=0.3),
        # one step of the full single-slice scan, 4096 positions
        _case("grad-2d-1024-m128", "grad", 128, 1, 1024, 1024, 64, 64, 14, strength=0.3),
        # one step of the 8-slice scan
        _case("grad-ms8-1024-m128", "grad", 128, 8, 1024, 1024, 64, 64, 14),
        # the 16-slice scan over 4 x 4 tiles, 16632 positions: the largest
        _case("tiles-ms16-2048-m128", "tiles", 128, 16, 2048, 2048, 126, 132, 14, ty=4, tx=4, halo=64),
        # autograd on an odd-sized object with a jittered scan: forward (loss) and backward (gradient)
        _case("train-ms3-odd-m128", "train", 128, 3, 389, 517, 17, 25, 14, jitter=3),
        # joint object and probe refinement
        _case("probe-ms4-640-m128", "probe", 128, 4, 640, 640, 31, 33, 14),
        # sub-pixel positions on a small multislice object
        _case("subpixel-ms2-m64", "subpixel", 64, 2, 300, 413, 27, 41, 8),
        # 32 independent reconstructions of uneven size, one captured gradient-descent iteration
        _case("batch32-uneven", "batch", 0, 0, 0, 0, 0, 0, 0, count=32, shapes=4, side=1024, raster=48),
        # neighbour addition and stitch of 4 x 4 tile gradients of 16 slices
        _case("exchange-ms16-2048", "exchange", 128, 16, 2048, 2048, 8, 8, 240, ty=4, tx=4, halo=64),
        # one iteration of the tiled reconstruction: 64 positions per tile between its updates
        _case("alg1-ms8-1024-m128", "alg1", 128, 8, 1024, 1024, 64, 64, 14, ty=2, tx=2, halo=64, batch=64, T=16),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["forward", "forward", "grad", "grad", "grad", "grad", "tiles", "train", "probe", "subpixel",
                       "batch", "exchange", "alg1"])
    M = rng.choice([64, 128])
    step = rng.randint(6, 11) if M == 64 else rng.randint(10, 18)
    jitter = rng.choice([0, 0, 1, 3])
    if kind == "batch":
        return _case(None, kind, 0, 0, 0, 0, 0, 0, 0, count=rng.randint(2, 32), shapes=rng.randint(0, 10 ** 6),
                     side=rng.choice([512, 768, 1024]), raster=rng.randint(10, 48))
    if kind in ("tiles", "exchange", "alg1"):
        M, S = 128, rng.choice([1, 2, 3, 4, 6, 8])
        ty, tx = rng.randint(2, 3), rng.randint(2, 4)
        H, W = rng.randint(140 * ty, 300 * ty), rng.randint(140 * tx, 300 * tx)
        more = {"ty": ty, "tx": tx, "halo": 64}
        if kind == "alg1":
            more.update(batch=rng.choice([8, 16, 33, 64, 100]), T=rng.choice([1, 2, 4]))
    else:
        S = rng.choice([1, 1, 2, 3, 4, 5, 8, 13, 16])
        if kind == "subpixel":
            S = min(S, 4)
        H, W = _log(rng, M + 3, 1200), _log(rng, M + 3, 1200)
        more = {}
    ny = rng.randint(1, max(1, min(64, (H - M - 2 * jitter) // step + 1)))
    nx = rng.randint(1, max(1, min(64, (W - M - 2 * jitter) // step + 1)))
    if M + (ny - 1) * step + 2 * jitter > H or M + (nx - 1) * step + 2 * jitter > W:
        jitter, ny, nx = 0, 1, 1
    return _case(None, kind, M, S, H, W, ny, nx, step, jitter, 10.0 ** rng.uniform(4, 6), 0.3 if S == 1 else 0.05, **more)


# ---------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------
def _gen(seed, k):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 1000003 + k)
    return g


def _phases(S, H, W, pitch, g):
    """S slices of unit Gaussians (sigma 1.5 px) on a jittered lattice, scaled to [0, 1]."""
    cy = torch.arange(pitch // 2, H, pitch, device=DEV)
    cx = torch.arange(pitch // 2, W, pitch, device=DEV)
    shape = (S, len(cy), len(cx))
    y = (cy[:, None] + torch.randint(-1, 2, shape, generator=g, device=DEV)).clamp_(0, H - 1)
    x = (cx[None, :] + torch.randint(-1, 2, shape, generator=g, device=DEV)).clamp_(0, W - 1)
    a = torch.zeros((S, H * W), device=DEV)
    a.scatter_(1, (y * W + x).reshape(S, -1), 1.0)
    ky = torch.exp(-2 * (math.pi * 1.5 * torch.fft.fftfreq(H, device=DEV)) ** 2)
    kx = torch.exp(-2 * (math.pi * 1.5 * torch.fft.rfftfreq(W, device=DEV)) ** 2)
    p = torch.fft.irfft2(torch.fft.rfft2(a.view(S, H, W)) * (ky[:, None] * kx), s=(H, W))
    lo, hi = p.amin((1, 2), keepdim=True), p.amax((1, 2), keepdim=True)
    return (p - lo) / (hi - lo)


def _probe(M, dose):
    R, C = (12.0, 2.0) if M == 64 else (20.0, 4.0)
    q = torch.fft.fftfreq(M, dtype=torch.float64, device=DEV) * M
    qq = torch.sqrt(q[:, None] ** 2 + q[None, :] ** 2)
    pupil = torch.where(qq <= R, torch.exp(-1j * C * (qq / R) ** 2), torch.zeros((), dtype=torch.complex128, device=DEV))
    p = torch.fft.fftshift(torch.fft.ifft2(pupil))
    return (p * math.sqrt(dose / (M * M)) / p.abs().square().sum().sqrt()).to(torch.complex64)


def _scan(case, g):
    M, step, j = case["M"], case["step"], case["jitter"]
    y = (case["H"] - (M + (case["ny"] - 1) * step)) // 2 + step * torch.arange(case["ny"], device=DEV)
    x = (case["W"] - (M + (case["nx"] - 1) * step)) // 2 + step * torch.arange(case["nx"], device=DEV)
    pos = torch.stack(torch.meshgrid(y, x, indexing="ij"), -1).reshape(-1, 2)
    if j:
        pos = pos + torch.randint(-j, j + 1, pos.shape, generator=g, device=DEV)
    return pos.to(torch.int32).contiguous()


def _propagator(M, dtype):
    f = torch.fft.fftfreq(M, PIXEL, dtype=torch.float64, device=DEV)
    return torch.exp(-1j * math.pi * WAVELENGTH * DZ * (f[:, None] ** 2 + f[None, :] ** 2)).to(dtype)


def _windows(obj, pos, M):
    """obj [S, H, W] as flat slices, and the flat indices [n, M, M] of the windows."""
    S, H, W = obj.shape
    r = torch.arange(M, device=DEV)
    p = pos.long()
    return obj.reshape(S, H * W), (p[:, 0, None, None] + r[:, None]) * W + (p[:, 1, None, None] + r)


def _far_field(obj, probes, pos, M, H, waves=None):
    flat, idx = _windows(obj, pos, M)
    psi = probes.expand(len(pos), M, M)
    for s in range(obj.shape[0]):
        if waves is not None:
            waves.append(psi)
        phi = psi * flat[s][idx]
        if s + 1 < obj.shape[0]:
            psi = torch.fft.ifft2(H * torch.fft.fft2(phi))
    return torch.fft.fft2(phi), idx


def _patterns(obj, probe, pos, M, dtype, out, chunk, shifted=None):
    H = _propagator(M, dtype)
    for i in range(0, len(pos), chunk):
        p = probe if shifted is None else _shift(probe, shifted[i:i + chunk])
        out[i:i + chunk] = _far_field(obj, p, pos[i:i + chunk], M, H)[0].abs().square()
    return out


def _shift(probe, d):
    """The probe translated by d pixels (Fourier shift theorem), one per row of d."""
    M = probe.shape[-1]
    q = torch.fft.fftfreq(M, dtype=torch.float64, device=DEV) * M
    d = d.double()
    ph = q[:, None] * d[:, 0, None, None] + q[None, :] * d[:, 1, None, None]
    return torch.fft.ifft2(torch.fft.fft2(probe) * torch.exp(-2j * math.pi * ph / M).to(probe.dtype))


def _inputs(case, seed):
    """Object (evaluation point), probe, positions, patterns and, for sub-pixel scans, the fractions."""
    M, S, H, W = case["M"], case["S"], case["H"], case["W"]
    g = _gen(seed, 1)
    pitch = 8 if M == 64 else 10
    phase = case["strength"] * _phases(S, H, W, pitch, g)
    eval_phase = phase + 0.01 * _phases(S, H, W, pitch, g)
    d = {"phase": eval_phase, "obj": torch.polar(torch.ones_like(phase), eval_phase), "probe": _probe(M, case["dose"]),
         "pos": _scan(case, g)}
    n = len(d["pos"])
    if case["kind"] == "subpixel":
        d["frac"] = torch.rand((n, 2), generator=g, device=DEV)
    if case["kind"] != "forward":
        truth = torch.polar(torch.ones_like(phase), phase)
        I = _patterns(truth, d["probe"], d["pos"], M, torch.complex64,
                      torch.empty((n, M, M), device=DEV), 512, d.get("frac"))
        d["meas"] = torch.poisson(I, generator=g)
    return d


def _step_size(d, M, S, H, W):
    """1 / (2 M^2 S max sum_i |P(r - r_i)|^2): the step of plain gradient descent."""
    cover = torch.zeros(H * W, dtype=torch.float64, device=DEV)
    p2 = d["probe"].to(torch.complex128).abs().square().reshape(-1)
    r = torch.arange(M, device=DEV)
    for p in d["pos"].long().split(2048):
        idx = ((p[:, 0, None, None] + r[:, None]) * W + p[:, 1, None, None] + r).reshape(len(p), -1)
        cover.index_add_(0, idx.reshape(-1), p2.repeat(len(p)))
    return 1.0 / (2.0 * M * M * S * float(cover.max()))


def _batch_cases(case):
    """The uneven reconstructions of a batch: sizes from the case alone."""
    rng = random.Random(case["shapes"])
    out = []
    for _ in range(case["count"]):
        M, S = rng.choice([64, 128]), rng.choice([1, 2, 4, 8])
        W = rng.choice([w for w in (256, 512, 768, 1024) if w <= case["side"]])
        step = round(M / 9)
        most = (W - M) // step + 1
        lo = min(8, case["raster"])
        ny, nx = (min(rng.randint(lo, case["raster"]), most) for _ in range(2))
        out.append(_case(None, "grad", M, S, W, W, ny, nx, step, dose=10.0 ** rng.uniform(4, 6)))
    return out


def _context(case, n):
    return pt.Context(case["M"], case["S"], *PHYSICS, max(n, 1))


def _plan(case, pos):
    return TileWalk(pos.cpu().numpy(), case["H"], case["W"], case["M"], (case["ty"], case["tx"]), case["halo"])


# ---------------------------------------------------------------------------------------------
# the calls
# ---------------------------------------------------------------------------------------------
def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind}
    if kind == "batch":
        recons = []
        for k, c in enumerate(_batch_cases(case)):
            d = _inputs(c, seed * 64 + k)
            recons.append(Recon(d["obj"], d["probe"], d["pos"], d["meas"], *PHYSICS,
                                _step_size(d, c["M"], c["S"], c["H"], c["W"])))
        st["batch"] = Batch(recons, history_rows=64)
        st["batch"].capture()
        return st
    if kind == "exchange":
        g = _gen(seed, 2)
        plan = _plan(case, _scan(case, g))
        walk = DecomposedTileWalk(_context(case, plan.n), plan)
        for b in walk.bufs:
            b.copy_(torch.randn(b.shape, dtype=b.dtype, generator=g, device=DEV))
        st.update(walk=walk, out=torch.empty((case["S"], case["H"], case["W"]), dtype=torch.complex64, device=DEV))
        return st
    d = _inputs(case, seed)
    n = len(d["pos"])
    st["ctx"] = _context(case, n)
    st.update(d)
    if kind == "forward":
        st["intens"] = torch.empty((n, case["M"], case["M"]), device=DEV)
        return st
    st["loss"] = torch.zeros(1, dtype=torch.float64, device=DEV)
    if kind in ("tiles", "alg1"):
        plan = _plan(case, d["pos"])
        st["meas"] = d["meas"][torch.from_numpy(plan.order).to(DEV)]
        if kind == "alg1":
            st["walk"] = Alg1Walk(st["ctx"], plan, d["obj"], d["probe"], st["meas"],
                                  _step_size(d, case["M"], case["S"], case["H"], case["W"]), case["batch"], case["T"])
            return st
        st["walk"] = AllTilesWalk(st["ctx"], plan)
    if kind == "train":
        st["V"] = d["phase"].requires_grad_()
        return st
    st["grad"] = torch.empty_like(d["obj"])
    if kind == "probe":
        st["probe_grad"] = torch.empty_like(d["probe"])
    if kind == "subpixel":
        st["probes"] = torch.empty((n, case["M"], case["M"]), dtype=torch.complex64, device=DEV)
    return st


def run(st):
    kind = st["kind"]
    if kind == "forward":
        return pt.ptycho_forward(st["ctx"], st["obj"], st["probe"], st["pos"], intens=st["intens"])
    if kind == "grad":
        loss, grad = pt.ptycho_loss_grad(st["ctx"], st["obj"], st["probe"], st["pos"], st["meas"], grad=st["grad"],
                                         loss=st["loss"])
        return {"loss": loss, "grad": grad}
    if kind == "probe":
        loss, grad = pt.ptycho_loss_grad(st["ctx"], st["obj"], st["probe"], st["pos"], st["meas"], grad=st["grad"],
                                         loss=st["loss"], probe_grad=st["probe_grad"])
        return {"loss": loss, "grad": grad, "probe_grad": st["probe_grad"]}
    if kind == "subpixel":
        probes = pt.ptycho_shift_probes(st["ctx"], st["probe"], st["frac"], out=st["probes"])
        loss, grad = pt.ptycho_loss_grad(st["ctx"], st["obj"], probes, st["pos"], st["meas"], grad=st["grad"],
                                         loss=st["loss"])
        return {"loss": loss, "grad": grad, "probes": probes}
    if kind == "train":
        st["V"].grad = None
        loss = amplitude_loss_potential(st["ctx"], st["V"], 1.0, st["probe"], st["pos"], st["meas"])
        loss.backward()
        return {"loss": loss.detach(), "grad": st["V"].grad}
    if kind == "tiles":
        loss = st["walk"].step(st["obj"], st["probe"], st["meas"], st["grad"])
        return {"loss": loss, "grad": st["grad"]}
    if kind == "batch":
        b = st["batch"]
        b.replay()
        return {"obj": [r.obj for r in b.recons], "grad": [r.grad for r in b.recons]}
    if kind == "exchange":
        walk = st["walk"]
        acc = walk.neighbour_add()
        stitch_interiors(walk.ctx, walk.plan, acc, st["out"])
        return {"acc": acc, "out": st["out"]}
    walk = st["walk"]
    return {"loss": walk.iteration(), "V": walk.V}


# ---------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------
def _position_flops(M, S, kind):
    """2D DFTs at 5 N log2 N and the pointwise work of one position."""
    N = M * M
    dft = 5.0 * N * math.log2(N)
    fwd = (2 * S - 1) * dft + (12 * S + 4) * N
    back = (2 * S - 1) * dft + (18 * S + 6) * N
    return {"forward": fwd, "train": 2 * fwd + back, "subpixel": fwd + back + 2 * dft}.get(kind, fwd + back)


def work(case):
    kind, M, S, H, W = (case[k] for k in ("kind", "M", "S", "H", "W"))
    if kind == "batch":
        parts = [work(c) for c in _batch_cases(case)]
        shift = sum(8 * c["S"] * c["H"] * c["W"] for c in _batch_cases(case))  # the updated object is written too
        return {"bytes": sum(p["bytes"] for p in parts) + shift, "flops": sum(p["flops"] for p in parts)}
    n, obj = case["ny"] * case["nx"], 8 * S * H * W
    if kind == "exchange":
        boxes = 0
        for a in range(case["ty"]):
            for b in range(case["tx"]):
                h = min((a + 1) * H // case["ty"] + case["halo"], H) - max(a * H // case["ty"] - case["halo"], 0)
                w = min((b + 1) * W // case["tx"] + case["halo"], W) - max(b * W // case["tx"] - case["halo"], 0)
                boxes += h * w
        return {"bytes": 2 * 8 * S * boxes + obj, "flops": 2 * S * 9 * boxes}
    flops = n * _position_flops(M, S, kind)
    data = n * M * M * 4 + 8 * M * M
    if kind == "subpixel":
        data += n * M * M * 8
    if kind == "train":
        return {"bytes": obj // 2 + 2 * data + obj // 2, "flops": flops}
    return {"bytes": data + (obj if kind == "forward" else 2 * obj), "flops": flops}


# ---------------------------------------------------------------------------------------------
# the same results in 64 bits, plain torch
# ---------------------------------------------------------------------------------------------
def _exact_loss_grad(obj, probe, pos, meas, M, grad, frac=None, probe_grad=None, chunk=128):
    """Adds dF/dRe t + i dF/dIm t into grad (complex128 [S, H, W]); returns F."""
    H = _propagator(M, torch.complex128)
    S = obj.shape[0]
    total = torch.zeros((), dtype=torch.float64, device=DEV)
    gflat = torch.view_as_real(grad).view(S, -1, 2)
    for i in range(0, len(pos), chunk):
        p = probe if frac is None else _shift(probe, frac[i:i + chunk])
        waves = []
        far, idx = _far_field(obj, p, pos[i:i + chunk], M, H, waves)
        mod = far.abs()
        diff = mod - meas[i:i + chunk].double().sqrt()
        total += diff.square().sum()
        chi = torch.fft.ifft2(torch.where(mod > 0, 2.0 * diff / mod, torch.zeros_like(mod)) * far) * (M * M)
        at = idx.reshape(-1)
        for s in range(S - 1, -1, -1):
            gflat[s].index_add_(0, at, torch.view_as_real(chi * waves[s].conj()).reshape(-1, 2))
            back = chi * obj[s].reshape(-1)[idx].conj()
            if s:
                chi = torch.fft.ifft2(H.conj() * torch.fft.fft2(back))
            elif probe_grad is not None:
                probe_grad += back.sum(0)
    return total


def _exact_alg1(case, d):
    M, S, H, W = case["M"], case["S"], case["H"], case["W"]
    step = _step_size(d, M, S, H, W)
    plan = _plan(case, d["pos"])
    order = torch.from_numpy(plan.order).to(DEV)
    pos, meas, probe = d["pos"][order], d["meas"][order], d["probe"].to(torch.complex128)
    boxes = [(p.box[0], p.box[0] + p.box[2], p.box[1], p.box[1] + p.box[3]) for p in plan.plans]
    V = [d["obj"][:, a:b, c:e].to(torch.complex128) for a, b, c, e in boxes]
    acc = [torch.zeros_like(v) for v in V]
    loss = torch.zeros(1, dtype=torch.float64, device=DEV)
    steps = max(-(-(p.hi - p.lo) // case["batch"]) for p in plan.plans)
    for j in range(steps):
        for k, p in enumerate(plan.plans):
            lo = p.lo + j * case["batch"]
            hi = min(p.hi, lo + case["batch"])
            if hi <= lo:
                continue
            g = torch.zeros_like(V[k])
            local = pos[lo:hi] - torch.tensor([p.box[0], p.box[1]], dtype=torch.int32, device=DEV)
            loss += _exact_loss_grad(V[k], probe, local, meas[lo:hi], M, g)
            acc[k] += g
            V[k] = V[k] - step * g
        if (j + 1) % case["T"] == 0 or j == steps - 1:
            total = torch.zeros((S, H, W), dtype=torch.complex128, device=DEV)
            for (a, b, c, e), x in zip(boxes, acc):
                total[:, a:b, c:e] += x
            for k, (a, b, c, e) in enumerate(boxes):
                V[k] = V[k] - step * total[:, a:b, c:e]
                acc[k].zero_()
    return {"loss": loss, "V": V}


def _exact_exchange(case, seed):
    st = prepare(case, seed)
    plan, bufs = st["walk"].plan, [b.to(torch.complex128) for b in st["walk"].bufs]
    ty, tx = plan.tiles
    out = torch.empty((case["S"], case["H"], case["W"]), dtype=torch.complex128, device=DEV)
    acc = []
    for k, p in enumerate(plan.plans):
        a = bufs[k].clone()
        for q in plan.plans:
            if q.index == k or abs(q.index // tx - k // tx) > 1 or abs(q.index % tx - k % tx) > 1:
                continue
            y0, y1 = max(p.box[0], q.box[0]), min(p.box[0] + p.box[2], q.box[0] + q.box[2])
            x0, x1 = max(p.box[1], q.box[1]), min(p.box[1] + p.box[3], q.box[1] + q.box[3])
            if y0 < y1 and x0 < x1:
                a[:, y0 - p.box[0]:y1 - p.box[0], x0 - p.box[1]:x1 - p.box[1]] += \
                    bufs[q.index][:, y0 - q.box[0]:y1 - q.box[0], x0 - q.box[1]:x1 - q.box[1]]
        t = p.tile
        out[:, t[0]:t[1], t[2]:t[3]] = a[:, t[0] - p.box[0]:t[1] - p.box[0], t[2] - p.box[1]:t[3] - p.box[1]]
        acc.append(a)
    return {"acc": acc, "out": out}


def exact(case, seed):
    kind, M = case["kind"], case["M"]
    if kind == "batch":
        objs, grads = [], []
        for k, c in enumerate(_batch_cases(case)):
            d = _inputs(c, seed * 64 + k)
            o = d["obj"].to(torch.complex128)
            g = torch.zeros_like(o)
            _exact_loss_grad(o, d["probe"].to(torch.complex128), d["pos"], d["meas"], c["M"], g)
            objs.append(o - _step_size(d, c["M"], c["S"], c["H"], c["W"]) * g)
            grads.append(g)
        return {"obj": objs, "grad": grads}
    if kind == "exchange":
        return _exact_exchange(case, seed)
    d = _inputs(case, seed)
    probe = d["probe"].to(torch.complex128)
    if kind == "forward":
        out = torch.empty((len(d["pos"]), M, M), dtype=torch.float64, device=DEV)
        return _patterns(d["obj"].to(torch.complex128), probe, d["pos"], M, torch.complex128, out, 128)
    if kind == "alg1":
        return _exact_alg1(case, d)
    if kind == "train":
        phase = d["phase"].double()
        obj = torch.polar(torch.ones_like(phase), phase)
    else:
        obj = d["obj"].to(torch.complex128)
    grad = torch.zeros_like(obj)
    pgrad = torch.zeros_like(probe) if kind == "probe" else None
    loss = _exact_loss_grad(obj, probe, d["pos"], d["meas"], M, grad, d.get("frac"), pgrad)
    if kind == "train":
        return {"loss": loss, "grad": (obj.conj() * grad).imag}
    out = {"loss": loss.reshape(1), "grad": grad}
    if kind == "probe":
        out["probe_grad"] = pgrad
    if kind == "subpixel":
        out["probes"] = torch.cat([_shift(probe, f) for f in d["frac"].split(512)])
    return out
