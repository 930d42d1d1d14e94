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
        assert "set_tiles" in logs[k][0]
    assert "memcpy async" in logs[2]  # the all-tiles gradient uploads its own table once
    assert all(x.startswith("launch ") for x in logs[4]), logs[4]


def test_alg1_tables_grow_and_stay():
    """More tiles than the table holds: it grows, at least to twice its size, and an outgrown table is not freed
    before the context (a captured launch may use it)."""
    out = host_hip.run(STATES + r'''
rc, h = context(64, 1, 100)
def run(ny, nx):
    tiles = states(1, list(boxes(64 * ny, 64 * nx, ny, nx, 1)))
    log()
    codes = [step(h, tiles, (c_int32 * (ny * nx + 1))(), 0), flush(h, tiles, ny, nx)]
    l = log()
    return codes, [x for x in l if not x.startswith("launch ")], sum("set_tiles" in x for x in l)
r = [run(64, 64), run(64, 65), run(70, 70), run(90, 91), run(64, 65)]
before = R.host_hip_used()
L.ptycho_destroy(h)
done(r=r, before=before, after=R.host_hip_used())
''')
    for (codes, _, _) in out["r"]:
        assert codes == [0, 0]
    assert [x for _, x, _ in out["r"]] == [[], ["malloc"], [], [], []]
    assert [n for _, _, n in out["r"]] == [2 * -(-k // 48) for k in (4096, 4160, 4900, 8190, 4160)]
    assert out["before"] > 0 and out["after"] == 0
