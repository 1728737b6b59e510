"""Source checks and starts with more sources than one block looks at (1,024), than
a start exchanges flags for unread (8,192) and than the check's blocks look at at
once (262,144): how many lie on obstacles, and the map of the free ones."""
import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

COUNTS = (1, 64, 256, 257, 1024, 1025, 2048, 8192, 8193, 70001, 262144, 262145, 1048576)


@pytest.mark.parametrize("n", COUNTS)
def test_sources_on_obstacles_are_counted(n):
    import paper_2004_00540_amd as omap
    rng = np.random.default_rng(n)
    occ = (rng.random((300, 417)) < 0.3).astype(np.uint8)
    free = np.argwhere(occ == 0).astype(np.int32)
    wall = np.argwhere(occ != 0).astype(np.int32)
    src = free[rng.integers(0, len(free), n)]
    dev = to_dev(occ)
    with omap.Plan(dev, src, src[:1]) as plan:
        for bad in sorted({1, n // 3, n}):
            if bad < 1:
                continue
            mixed = src.copy()
            mixed[rng.permutation(n)[:bad]] = wall[rng.integers(0, len(wall), bad)]
            with pytest.raises(omap.OmapError, match=f" {bad} source") as e:
                plan.load(dev, mixed, src[:1])
            assert e.value.name == "OMAP_ERR_SOURCE_ON_OBSTACLE"
            with pytest.raises(omap.OmapError, match=f" {bad} source"):
                omap.Plan(dev, mixed, src[:1])
        plan.load(dev, src, src[:1])
        info = plan.propagate()
        d, ecc = oracle.bfs(occ, src)
        A = oracle.activity_from_bfs(d, ecc)
        assert info["layers"] == ecc and info["reached_cells"] == int((A > 0).sum())
        assert np.array_equal(plan.activity().cpu().numpy(), A)


@pytest.mark.parametrize("schedule", [0, 1, 2])
@pytest.mark.parametrize("layers", [-1, 0, 9])
def test_sources_of_many_mazes(schedule, layers):
    """Seeds of several mazes in one wave, repeated sources among them: each counted once."""
    import paper_2004_00540_amd as omap
    rng = np.random.default_rng(17)
    mazes, refs = [], []
    for n in (1, 2, 3, 30, 64, 1, 63, 500, 1, 1, 129, 5):
        occ = (rng.random((int(rng.integers(1, 150)), int(rng.integers(1, 200)))) < 0.3).astype(np.uint8)
        occ[0, 0] = 0
        free = np.argwhere(occ == 0).astype(np.int32)
        src = free[rng.integers(0, max(1, len(free) // 2), n)]
        d, ecc = oracle.bfs(occ, src)
        mazes.append((to_dev(occ), src, src[:1]))
        refs.append((ecc if layers < 0 else layers, oracle.activity_from_bfs(d, ecc if layers < 0 else layers)))
    with omap.Batch(mazes, schedule=schedule) as b:
        for _ in range(2):
            for i, info in enumerate(b.propagate([layers] * len(mazes))):
                assert (info["layers"], info["reached_cells"]) == (refs[i][0], int((refs[i][1] > 0).sum())), i
                assert np.array_equal(b.activity(i).cpu().numpy(), refs[i][1]), i
