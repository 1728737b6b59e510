"""Packing of the occupancy: widths around a lane's 16 bytes, a word's 32 columns
and a block's 1024, heights around a wave's eight rows and a block's 32, obstacle
bytes of every value, odd addresses, both mask layouts, one maze and several."""
import numpy as np
import pytest

import workloads
from gpu_helpers import oracle_solution

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (9, 15), (7, 16), (8, 17), (31, 31), (33, 33), (65, 47), (32, 1023), (33, 1024), (34, 1041)]


def _maze(H, W):
    """A random maze and the same with obstacles as bytes 1 .. 255."""
    m = workloads.random_maze(H, W, 0.3, 3, 4, 6200 + 5 * H + W)
    values = np.random.default_rng(W).integers(1, 256, m.occ.shape).astype(np.uint8)
    return m, np.where(m.occ != 0, values, 0).astype(np.uint8)


def _at(occ, offset):
    import torch
    flat = torch.zeros(offset + occ.size, dtype=torch.uint8, device="cuda")
    flat[offset:] = torch.from_numpy(occ).cuda().flatten()
    return flat[offset:].view(occ.shape)


OPTIONS = [{}, {"schedule": 1, "temporal_depth": 8}]     # strips; rows (the integer sweep's layout)


@pytest.mark.parametrize("options", OPTIONS)
@pytest.mark.parametrize("shape", SHAPES)
def test_pack_one(shape, options):
    import paper_2004_00540_amd as omap
    m, occ = _maze(*shape)
    A = oracle_solution(m, -1)[0]
    for offset in (0, 1, 7):
        with omap.Plan(_at(occ, offset), m.sources, m.targets, **options) as plan:
            plan.propagate()
            assert np.array_equal(plan.activity().cpu().numpy(), A), (shape, offset)


@pytest.mark.parametrize("options", OPTIONS)
def test_pack_several(options):
    import paper_2004_00540_amd as omap
    ms = [_maze(*s) for s in SHAPES]
    with omap.Batch([(_at(occ, i % 3), m.sources, m.targets) for i, (m, occ) in enumerate(ms)], **options) as b:
        b.propagate()
        for i, (m, _) in enumerate(ms):
            assert np.array_equal(b.activity(i).cpu().numpy(), oracle_solution(m, -1)[0]), (i, m.occ.shape)
