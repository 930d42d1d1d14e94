"""What the library's host side asks of the HIP runtime -- launches, allocations, copies, waits -- followed
without a GPU on a runtime that records (host_hip)."""
import host_hip

STATES = r'''
def states(S, bx):
    return (State * len(bx))(*[State(*b, *[device(S * b[6] * b[7] * 8) for _ in range(3)]) for b in bx])
def step(h, tiles, seg, lists):
    n = len(tiles)
    dev = [device(4 << 20) for _ in range(7)]
    return L.ptycho_tiles_batch_step(h, tiles, n, *dev[:4], lists, dev[4], seg[n], dev[5], seg, c_float(0.1), dev[6])
def flush(h, tiles, ny, nx):
    return L.ptycho_tiles_flush(h, tiles, ny, nx, c_float(0.1))
'''


def test_alg1_calls_only_launch():
    """A batch and a flush, first ones included and with other tile calls on the context in between, consist of
    launches: no wait, copy or allocation, so they can be captured at any time."""
    out = host_hip.run(STATES + r'''
rc, h = context(64, 2, 100)
bx = list(boxes(256, 256, 2, 2, 32))
one, two = states(2, bx), states(2, bx)
tiles = (Tile * 4)(*[Tile(*b, device(2 * b[6] * b[7] * 8)) for b in bx])
seg = (c_int32 * 5)(0, 2, 4, 6, 8)
d = [device(4 << 20) for _ in range(7)]
grad = lambda: L.ptycho_tiles_grad(h, d[0], 256, 256, c_int64(256 * 256), 256, tiles, 4, 32, d[1], d[2], d[3], 8, d[4],
                                   d[5], None, 0)
codes, logs = [rc], []
log()
for call in (lambda: step(h, one, seg, 8), lambda: flush(h, one, 2, 2), grad, lambda: step(h, two, seg, 8), grad,
             lambda: flush(h, one, 2, 2)):
    codes.append(call())
    logs.append(log())
done(codes=codes, logs=logs)
''')
    assert out["codes"] == [0] * 7
    logs = out["logs"]
    for k in (0, 1, 3, 5):
        assert logs[k] and all(x.startswith("launch ") for x in logs[k]), logs[k]
    assert len(logs[0]) == len(logs[3]) == 2  # gradient and update: few tiles travel in their arguments
    assert "memcpy async" in logs[2]  # the all-tiles gradient uploads its own table once
    assert all(x.startswith("launch ") for x in logs[4]), logs[4]


def test_alg1_tables_grow_and_stay():
    """More than 48 tiles go through the context's table, 48 to a launch; the gradient stays one launch.  More
    than the table holds: it grows, at least to twice its size, and an outgrown table is not freed before the
    context (a captured launch may use it)."""
    out = host_hip.run(STATES + r'''
rc, h = context(64, 1, 100)
def run(ny, nx):
    n = ny * nx
    tiles = states(1, list(boxes(64 * ny, 64 * nx, ny, nx, 1)))
    log()
    codes = [step(h, tiles, (c_int32 * (n + 1))(0, *[1] * n), 1), flush(h, tiles, ny, nx)]
    l = log()
    return codes, [x for x in l if not x.startswith("launch ")], [sum(k in x for x in l) for k in (
        "set_tiles", "fused_kernel", "tile_step", "tile_flush")]
r = [run(8, 6), run(7, 7), run(64, 64), run(64, 65), run(70, 70), run(90, 91), run(64, 65)]
before = R.host_hip_used()
L.ptycho_destroy(h)
done(r=r, before=before, after=R.host_hip_used())
''')
    for (codes, _, _) in out["r"]:
        assert codes == [0, 0]
    assert [x for _, x, _ in out["r"]] == [[], [], [], ["malloc"], [], [], []]
    parts = [-(-k // 48) for k in (48, 49, 4096, 4160, 4900, 8190, 4160)]
    assert [n for _, _, n in out["r"]] == [[p if p > 1 else 0, 1, p, p] for p in parts]
    assert out["before"] > 0 and out["after"] == 0


def test_stores_fit_the_capacity():
    """64-window contexts hold stores for three workgroups per CU, 128-windows for one; a context whose gradient
    calls cannot use more than one per CU holds no more, until reserve raises the capacity.  Pattern launches,
    which need no store, take the whole device either way."""
    out = host_hip.run(r'''
def forward(h, M, n):
    log()
    rc = L.ptycho_forward(h, device(1 << 20), 256, 256, c_int64(1 << 16), 256, device(1 << 17), device(1 << 20), n,
                          device(4 * n * M * M))
    return rc, log()
def grad(h, M, n, probe_grad):
    log()
    d = [device(1 << 20) for _ in range(8)]
    rc = L.ptycho_loss_grad_probe(h, d[0], 256, 256, c_int64(1 << 16), 256, d[1], d[2], n, d[3], d[4], None, d[5],
                                  c_int64(1 << 16), 256, d[6] if probe_grad else None, 0, None)
    return rc, [x for x in log() if "fused_kernel" in x]
r = {}
for name, M, capacity in (("one", 64, 1), ("cus", 64, 256), ("more", 64, 257), ("large", 128, 5000)):
    rc, h = context(M, 5, capacity)
    r[name] = [rc, L.ptycho_workspace_bytes(h), forward(h, M, 5000), grad(h, M, min(capacity, 5000), True)]
    assert L.ptycho_workspace_bytes(h) == R.host_hip_used()
    if name == "one":
        r["reserve"] = [L.ptycho_reserve(h, 5000), L.ptycho_workspace_bytes(h), grad(h, M, 5000, False)]
        r["interval"] = [L.ptycho_set_checkpoint(h, 2), L.ptycho_workspace_bytes(h), grad(h, M, 5000, False)]
        assert L.ptycho_workspace_bytes(h) == R.host_hip_used()
    L.ptycho_destroy(h)
    assert R.host_hip_used() == 0
done(**r)
''')
    slot = 64 * 64 * 8
    tables = out["one"][1] - 256 * 5 * slot
    assert 0 < tables < 1 << 20
    assert out["cus"][1] == 256 * 5 * slot + tables + 8 * 255
    assert out["more"][1] == 768 * 5 * slot + tables + 8 * 256
    assert out["large"][1] == 256 * 5 * 4 * slot + tables + 8 * 4999 + 2 * 8 * 64
    for name, wide, launched in (("one", 768, 1), ("cus", 768, 256), ("more", 768, 257), ("large", 256, 256)):
        rc, _, (rc_f, forward), (rc_g, grad) = out[name]
        assert rc == rc_f == rc_g == 0
        assert f" grid {wide} 1 1 " in forward[0] and f" grid {launched} 1 1 " in grad[0]
    rc, total, (rc_g, grad) = out["reserve"]
    assert rc == rc_g == 0 and " grid 768 1 1 " in grad[0]
    assert total == 768 * 5 * slot + tables + 8 * 4999
    rc, total, (rc_g, grad) = out["interval"]  # S = 5, interval 2: two checkpoints, an inner and the parked wave
    assert rc == rc_g == 0 and " grid 768 1 1 " in grad[0]
    assert total == 768 * (4 + 1) * slot + tables + 8 * 4999


def test_contexts_fit_where_one_workgroup_per_cu_fits():
    """Whatever the room, a context comes up where the stores of one workgroup per CU fit, and changes its
    checkpoint interval where the new store fits beside the old one; a refusal leaves it as it was."""
    out = host_hip.run(r'''
slot = 64 * 64 * 8
rc, h = context(64, 9, 300)
full = L.ptycho_workspace_bytes(h)
L.ptycho_destroy(h)
small = full - 512 * 9 * slot
r = []
for k in range(0, 21):
    room = small + (full - small) * k // 20 + (k // 20) * 4096 - (0 if k else 1)
    budget(room)
    rc, h = context(64, 9, 300)
    r.append([rc, L.ptycho_workspace_bytes(h) if rc == 0 else R.host_hip_used()])
    if rc == 0: L.ptycho_destroy(h)
    assert R.host_hip_used() == 0
budget(full)
_, h = context(64, 9, 300)
assert L.ptycho_set_checkpoint(h, 3) == -8 and L.ptycho_workspace_bytes(h) == full  # no room beside the old one
budget(full + 256 * 5 * slot)
c = [L.ptycho_set_checkpoint(h, 3), L.ptycho_workspace_bytes(h), R.host_hip_used()]
done(r=r, full=full, small=small, c=c)
''')
    assert out["r"][0] == [-8, 0]
    assert all(rc == 0 for rc, _ in out["r"][1:])
    assert all(b == out["small"] for _, b in out["r"][1:20]) and out["r"][20][1] == out["full"]
    # interval 3 for one workgroup per CU: two checkpoints, two inner waves and the parked one; the probe
    # partials stay
    after = out["full"] - (768 * 8 - 256 * 5) * 32768
    assert out["c"] == [0, after, after]


def test_a_stitch_of_many_tiles_costs_the_host_no_more_than_the_boxes():
    """4096 tiles, as a grid and as strips: finding the boxes over each tile takes the host no longer than
    twice the calls that add box by box (all pairs of tiles took eight times as long)."""
    out = host_hip.run(r'''
import time
r = []
for H, W, ny, nx, halo in ((4096, 4096, 64, 64, 32), (64, 65536, 1, 4096, 8), (65536, 64, 4096, 1, 8)):
    rc, h = context(64, 1, 16)
    bx = list(boxes(H, W, ny, nx, halo))
    tiles = (Tile * len(bx))(*[Tile(*b, device(b[6] * b[7] * 8)) for b in bx])
    dst = device(H * W * 8)
    best = [1e9, 1e9]
    for _ in range(3):
        t = time.perf_counter()
        rc |= L.ptycho_tiles_stitch(h, tiles, len(bx), H, W, dst, c_int64(H * W), W, 0)
        best[0] = min(best[0], time.perf_counter() - t)
        t = time.perf_counter()
        for b, k in zip(bx, tiles):
            rc |= L.ptycho_tile_accumulate(h, c_void_p(k.grad), b[4], b[5], b[6], b[7], H, W, dst, c_int64(H * W), W)
        best[1] = min(best[1], time.perf_counter() - t)
        R.host_hip_clear()
    r.append([rc] + best)
done(r=r)
''')
    for rc, stitch, by_box in out["r"]:
        assert rc == 0 and stitch <= 2 * by_box, out


def test_runs_of_positions_by_launch():
    """Runs of 8 consecutive positions per workgroup for gradients, whatever the size of the object and also
    for Alg. 1's batches; 2 for the all-tiles launch when object and boxes exceed 1 GiB, and without a gradient
    for objects over 128 MiB; one whole run for the register sums."""
    out = host_hip.run(STATES + r'''
def runs():
    return [int(x.split(" run ")[1]) for x in log() if "fused_kernel" in x]
r = {}
def objects(name, M, S, W):
    rc, h = context(M, S, 5000)
    log()
    d = [device(8 * S * W * W + (1 << 20)) for _ in range(6)]
    args = (h, d[0], W, W, c_int64(W * W), W, d[1], d[2], 5000, d[3])
    rc |= L.ptycho_loss_grad(*args, d[4], None, d[5], c_int64(W * W), W, 0, None)
    rc |= L.ptycho_loss(*args, d[4], None, 0)
    rc |= L.ptycho_forward(*args[:9], d[5])
    r[name] = [rc] + runs()
def tiles(name, S, W, n):
    rc, h = context(128, S, 5000)
    bx = list(boxes(W, W, n, n, 64))
    t = (Tile * (n * n))(*[Tile(*b, device(8 * S * b[6] * b[7])) for b in bx])
    d = [device(8 * S * W * W + (1 << 20)) for _ in range(6)]
    log()
    rc |= L.ptycho_tiles_grad(h, d[0], W, W, c_int64(W * W), W, t, n * n, 64, d[1], d[2], d[3], 5000, d[4], d[5], None,
                              0)
    s = states(S, bx)
    seg = (c_int32 * (n * n + 1))(*[5000 * k // (n * n) for k in range(n * n + 1)])
    rc |= step(h, s, seg, 5000)
    r[name] = [rc] + runs()
objects("small", 128, 8, 512)
objects("large", 128, 8, 4096)
objects("sums", 64, 1, 512)
tiles("few", 8, 1024, 2)
tiles("many", 16, 2048, 4)
done(**r)
''')
    assert out == {"small": [0, 8, 8, 8], "large": [0, 8, 2, 2], "sums": [0, 1 << 20, 8, 8], "few": [0, 8, 8],
                   "many": [0, 2, 8]}


def test_alg1_calls_refuse_bad_arguments():
    """The batch step and the flush check their tiles, segments and sizes on the host and enqueue nothing when
    they refuse."""
    out = host_hip.run(STATES + r'''
rc, h = context(64, 2, 10)
bx = list(boxes(256, 256, 2, 2, 32))
good = states(2, bx)
dev = [device(4 << 20) for _ in range(7)]
def call(tiles=good, n=4, lists=8, seg=(0, 2, 4, 6, 8), step=0.1, total=100, null=None, ctx=h):
    a = [None if i == null else p for i, p in enumerate(dev)]
    s = (c_int32 * len(seg))(*seg) if seg else None
    return L.ptycho_tiles_batch_step(ctx, tiles, n, a[0], a[1], a[2], a[3], total, a[4], lists, a[5], s, c_float(step),
                                     a[6])
def flush(tiles=good, ny=2, nx=2, step=0.1, ctx=h):
    return L.ptycho_tiles_flush(ctx, tiles, ny, nx, c_float(step))
def changed(k, **fields):
    t = states(2, bx)
    for f, v in fields.items():
        setattr(t[k], f, v)
    return t
log()
inf = float("inf")
r = dict(
    context=call(ctx=None), tiles=call(tiles=None), none=call(n=0), step=call(step=inf),
    total=call(total=-1), negative=call(lists=-1),
    capacity=call(lists=11, seg=(0, 2, 4, 6, 11)), segments=call(seg=None), short=call(seg=(0, 2, 4, 6, 7)),
    first=call(seg=(1, 2, 4, 6, 8)), decrease=call(seg=(0, 4, 2, 6, 8)),
    nulls=[call(null=i) for i in range(7)],
    shared=call(tiles=changed(1, acc=good[1].acc, grad=good[1].acc)),
    overlap=call(tiles=changed(2, obj=good[2].obj + 8, acc=good[2].obj)),
    buffer=call(tiles=changed(0, acc=None)), outside=call(tiles=changed(0, ty0=-1)), box=call(tiles=changed(0, eh=0)),
    far=call(tiles=changed(0, ey0=2**31 - 10, ty0=2**31 - 10, ty1=2**31 - 1)),
    small=call(tiles=changed(3, ey0=192, ty0=192, ty1=255, eh=63)),
    flush=[flush(ctx=None), flush(tiles=None), flush(ny=0), flush(nx=70000), flush(step=-inf),
           flush(tiles=changed(1, grad=good[1].obj, obj=good[1].obj))])
l = log()
ok = [call(lists=0, seg=(0,) * 5), call(), flush(),
      call(tiles=changed(3, ey0=192, ty0=192, ty1=255, eh=63), lists=6, seg=(0, 2, 4, 6, 6))]
done(log=l, ok=ok, launches=len(log()), **r)
''')
    arg, shape, halo, capacity = -1, -2, -4, -9
    assert out["log"] == []
    assert out["ok"] == [0] * 4 and out["launches"] > 0
    for name in ("context", "tiles", "none", "step", "total", "negative", "segments", "short", "first", "decrease",
                 "shared", "overlap", "buffer"):
        assert out[name] == arg, name
    assert out["nulls"] == [arg] * 7 and out["flush"] == [arg] * 6
    assert out["capacity"] == capacity and out["small"] == halo
    assert out["outside"] == out["box"] == out["far"] == shape
