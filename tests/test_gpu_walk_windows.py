"""Random-tie and Euclidean walks where they cross windows of the map (48 x 64
cells), groups of 64 random numbers and of 64 stored points, and where every
move has ties: serpentine mazes, open maps and a maze without 4-neighbour
moves, against the oracle."""
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


def _mazes():
    out = []
    for H, W in ((20, 30), (39, 57), (121, 203), (5, 300)):
        occ = _serpentine(H, W)
        free = np.argwhere(occ == 0).astype(np.int32)
        out.append(workloads.Maze(occ, free[:1], free[::7].copy(), f"serpentine {H}x{W}"))
        out.append(workloads.Maze(np.ascontiguousarray(occ.T), free[:1, ::-1].copy(), free[::7, ::-1].copy(), f"serpentine {W}x{H}"))
    open_map = np.zeros((150, 260), np.uint8)      # up to three maximal neighbours at every move
    cells = np.argwhere(open_map == 0).astype(np.int32)
    out.append(workloads.Maze(open_map, np.array([[75, 130], [0, 259]], np.int32), cells[::61].copy(), "open"))
    diag = np.ones((200, 200), np.uint8)           # a diagonal corridor: only the 8-neighbour fallback moves
    diag[np.arange(200), np.arange(200)] = 0
    on = np.stack([np.arange(200)] * 2, 1).astype(np.int32)
    out.append(workloads.Maze(diag, on[:1], on[::9].copy(), "diagonal"))
    out.append(workloads.random_maze(333, 517, 0.38, 2, 60, 515))
    return out


@pytest.mark.parametrize("mode", ["random", "euclidean"])
@pytest.mark.parametrize("layers", [-1, 190])
def test_walk_windows(mode, layers):
    import paper_2004_00540_amd as omap
    for m in _mazes():
        d, ecc = oracle.bfs(m.occ, m.sources)
        A = oracle.activity_from_bfs(d, ecc if layers < 0 else layers)
        print(m.name, mode, layers, flush=True)
        ref = (oracle.walk_random(A, m.sources, m.targets, 12345) if mode == "random"
               else oracle.walk_euclidean(A, m.sources, m.targets))
        with omap.Plan(to_dev(m.occ), m.sources, m.targets) as plan:
            plan.propagate(layers)
            got = [t.cpu().numpy() for t in plan.paths(mode, 12345)]
        for g, r in zip(got, ref):
            assert np.array_equal(g, r), (m.name, mode, layers)
