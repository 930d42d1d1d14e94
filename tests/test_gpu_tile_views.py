"""Tile buffers that share memory: what the per-box calls take, the whole-grid ones must not refuse."""
import numpy as np
import pytest

import paper_2205_06327_amd as pt
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
