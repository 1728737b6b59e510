"""Paths followed by a block per target (few targets, long paths) and by a wave per
target (others): windows of 64 x 64 cells, 8 moves a hop, maps narrower than a
window, long winding and straight paths, ties at every move."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


def _serpentine(H, W):
    occ = np.zeros((H, W), np.uint8)
    for k, r in enumerate(range(1, H - 1, 2)):
        occ[r, :] = 1
        occ[r, W - 1 if k % 2 == 0 else 0] = 0
    return occ


def _maps():
    diag = np.ones((200, 200), np.uint8)
    diag[np.arange(200), np.arange(200)] = 0
    yield "serpentine", _serpentine(121, 203), 1
    yield "serpentine down", np.ascontiguousarray(_serpentine(131, 67).T), 1
    yield "diagonal", diag, 1
    yield "open", np.zeros((150, 260), np.uint8), 3
    for H, W in ((1, 1), (1, 300), (300, 1), (2, 63), (62, 62), (64, 65), (333, 517)):
        yield f"random {H}x{W}", workloads.random_maze(H, W, 0.3, 2, 4, 900 + H + W).occ, 2


@pytest.mark.parametrize("n", [1, 256, 257, 512, 513])
def test_walk_tile(n):
    import paper_2004_00540_amd as omap
    for name, occ, n_sources in _maps():
        free = np.argwhere(occ == 0).astype(np.int32)
        rng = np.random.default_rng(n + len(free))
        src = free[rng.permutation(len(free))[:n_sources]]
        if name.startswith(("serp", "diag")):
            src = free[:1]
        tgt = free[rng.integers(0, len(free), n)]
        tgt[0] = free[-1]
        d, ecc = oracle.bfs(occ, src)
        for layers in (-1, 190):
            A = oracle.activity_from_bfs(d, ecc if layers < 0 else layers)
            print(name, n, layers, flush=True)
            ref = oracle.walk(A, src, tgt)
            with omap.Plan(to_dev(occ), src, tgt) as plan:
                plan.propagate(layers)
                got = [g.cpu().numpy() for g in plan.paths()]
            for g, r in zip(got, ref):
                assert np.array_equal(g, r), (name, n, layers)
