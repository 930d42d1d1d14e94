"""Tile buffers that share memory, and tiles that are no grid: what the per-box calls take, the whole-grid
ones must not refuse or sum another way."""
import numpy as np
import pytest

import paper_2205_06327_amd as pt
from paper_2205_06327_amd import _binding as B
from paper_2205_06327_amd.tilewalk import TileWalk, neighbour_add

from gpu_helpers import say

pytestmark = pytest.mark.gpu


def test_neighbour_add_reads_overlapping_sources():
    """The sources are only read and may be overlapping views of one array: full-width rows of a single slice
    are contiguous without a copy."""
    import torch
    H, W = 190, 150
    say("neighbour addition of overlapping row views")
    plan = TileWalk(np.zeros((1, 2), np.int32), H, W, 64, (3, 1), 16)
    ctx = pt.Context(64, 1, 0.0197, 2.0, 0.1, 16)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    whole = torch.randn((1, H, W), dtype=torch.complex64, generator=g, device="cuda:0")
    views = [whole[:, p.box[0]:p.box[0] + p.box[2]] for p in plan.plans]
    assert all(v.is_contiguous() for v in views)
    got, want = [torch.empty_like(v) for v in views], [torch.empty_like(v) for v in views]
    neighbour_add(ctx, plan, views, got)
    neighbour_add(ctx, plan, [v.clone() for v in views], want)
    for a, b in zip(got, want):
        assert torch.equal(a, b)


def _cut(rng, rect, depth):
    """A rectangle (y0, y1, x0, x1) cut at random, again and again."""
    y0, y1, x0, x1 = rect
    if depth == 0 or max(y1 - y0, x1 - x0) < 4:
        return [rect]
    if y1 - y0 > x1 - x0 or (rng.random() < 0.4 and y1 - y0 > 3):
        m = int(rng.integers(y0 + 1, y1))
        parts = [(y0, m, x0, x1), (m, y1, x0, x1)]
    else:
        m = int(rng.integers(x0 + 1, x1))
        parts = [(y0, y1, x0, m), (y0, y1, m, x1)]
    return [t for p in parts for t in _cut(rng, p, depth - 1)]


@pytest.mark.parametrize("H,W,depth,halo,empty", [(90, 310, 6, 17, 0), (300, 41, 7, 5, 3), (128, 128, 3, 0, 0),
                                                  (64, 64, 5, 64, 2)])
def test_stitch_of_uneven_tiles(H, W, depth, halo, empty):
    """Tiles cut at random, in any order, some of them empty (their boxes still count): the stitch equals the
    boxes added one after another, bit for bit."""
    import torch
    say(f"stitch of uneven tiles, {H}x{W}, depth {depth}, halo {halo}")
    rng = np.random.default_rng(H)
    rects = _cut(rng, (0, H, 0, W), depth) + [(int(y), int(y), int(x), int(x) + 2) for y, x in
                                              rng.integers(1, min(H, W) - 2, (empty, 2))]
    rects = [rects[k] for k in rng.permutation(len(rects))]
    ctx = pt.Context(64, 2, 0.0197, 2.0, 0.1, 16)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(9)
    tiles = []
    for y0, y1, x0, x1 in rects:
        ey0, ey1, ex0, ex1 = max(y0 - halo, 0), min(y1 + halo, H), max(x0 - halo, 0), min(x1 + halo, W)
        box = (ey0, ex0, max(ey1 - ey0, 1), ex1 - ex0)
        tiles.append(((y0, y1, x0, x1), box, torch.randn((2, box[2], box[3]), dtype=torch.complex64, generator=g,
                                                         device="cuda:0")))
    want = torch.zeros((2, H, W), dtype=torch.complex64, device="cuda:0")
    got = torch.empty_like(want)
    for _, box, b in tiles:
        B.ptycho_tile_accumulate(ctx, b, box, want)
    B.ptycho_tiles_stitch(ctx, tiles, got)
    assert torch.equal(got, want)
    inner = torch.empty_like(want)
    B.ptycho_tiles_stitch(ctx, tiles, inner, B.STITCH_INTERIOR)
    for (y0, y1, x0, x1), (ey0, ex0, _, _), b in tiles:
        assert torch.equal(inner[:, y0:y1, x0:x1], b[:, y0 - ey0:y1 - ey0, x0 - ex0:x1 - ex0])
    wrong = [((y0, y1, x0, x1), box, b) for (y0, y1, x0, x1), box, b in tiles]
    k = next(i for i, t in enumerate(wrong) if t[0][1] > t[0][0] and t[0][0] > 0)
    (y0, y1, x0, x1), box, b = wrong[k]
    if box[0] < y0:  # one row into its neighbour
        wrong[k] = ((y0 - 1, y1 - 1, x0, x1), box, b)
        with pytest.raises(pt.PtychoError) as e:
            B.ptycho_tiles_stitch(ctx, wrong, got)
        assert e.value.name == "PTYCHO_E_SHAPE"
