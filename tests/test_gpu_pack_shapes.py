"""Packing of mazes narrower than a block's 32 words and lower than its 32 rows:
every power of two of rows and words to a block and one beside it, alone and among
many others, both mask layouts."""
import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

HEIGHTS = (1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 63, 129, 256, 257, 511, 512, 513, 1025)
WIDTHS = (1, 8, 15, 16, 17, 64, 65, 128, 129, 256, 257, 512, 513, 1024, 1025)


def _maze(H, W):
    rng = np.random.default_rng(H * 2000 + W)
    occ = np.where(rng.random((H, W)) < 0.25, rng.integers(1, 256, (H, W)), 0).astype(np.uint8)
    src = np.stack([rng.integers(0, H, 5), rng.integers(0, W, 5)], 1).astype(np.int32)
    occ[src[:, 0], src[:, 1]] = 0
    d, ecc = oracle.bfs(occ, src)
    return occ, src, oracle.activity_from_bfs(d, ecc)


@pytest.mark.parametrize("options", [{}, {"schedule": 1, "temporal_depth": 8}])
@pytest.mark.parametrize("H", HEIGHTS)
def test_pack_low_and_narrow(H, options):
    import paper_2004_00540_amd as omap
    mazes = [_maze(H, W) for W in WIDTHS]
    items = [(to_dev(occ), src, None) for occ, src, _ in mazes]
    for (occ, src, _), (_, _, A) in zip(items, mazes):
        with omap.Plan(occ, src, **options) as plan:
            plan.propagate()
            assert np.array_equal(plan.activity().cpu().numpy(), A), A.shape
    with omap.Batch(items * 5, **options) as b:
        b.propagate()
        for i in range(len(b)):
            assert np.array_equal(b.activity(i).cpu().numpy(), mazes[i % len(mazes)][2]), (i, b.shapes[i])


@pytest.mark.parametrize("H,W", [(1, 4000000), (3, 1000003), (4000000, 1), (1000003, 9), (70000, 65)])
def test_pack_long_and_thin(H, W):
    import paper_2004_00540_amd as omap
    occ, src, _ = _maze(H, W)
    d, _ = oracle.bfs(occ, src)
    A = oracle.activity_from_bfs(d, 300)
    with omap.Plan(to_dev(occ), src) as plan:
        plan.propagate(300)
        assert np.array_equal(plan.activity().cpu().numpy(), A)
