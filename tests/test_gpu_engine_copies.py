"""Host copies of the engine that are split over worker threads: sizes that a chunk
size rounded down leaves bytes of (an odd number of them over multiples of 64)."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import oracle
import workloads
from gpu_helpers import oracle_solution

pytestmark = pytest.mark.gpu


def _solve(eng, *args):
    import paper_2004_00540_amd as omap
    qid = eng.submit(*args)
    for _ in range(20000):
        eng.step(rounds=40)
        if eng.poll(qid) in (omap.QUERY_DONE, omap.QUERY_FAILED):
            break
    assert eng.poll(qid) == omap.QUERY_DONE
    return eng.fetch(qid)


@pytest.mark.parametrize("H,W", [(387, 5419), (1, 3145729), (1, 4194307), (2048, 2048)])   # 2, 3, 4, 4 chunks
def test_last_cells_of_a_grid_arrive(H, W):
    import paper_2004_00540_amd as omap
    occ = np.zeros((H, W), np.uint8)
    with omap.Engine(1 << 30, max_slots=1) as eng:
        for last in (0, 1, 0, 7):           # the pinned copy's place holds the grid before
            occ[-1, -1] = last
            L = 40
            src = np.array([[H - 1, W - 8]], np.int32)
            got = _solve(eng, occ, src, np.array([[H - 1, W - 1]], np.int32), L)
            d, _ = oracle.bfs(occ, src)
            A = oracle.activity_from_bfs(d, L)
            assert got.info["reached_cells"] == int((A > 0).sum()), last
            assert (got.lengths[0] >= 0) == (last == 0)


@pytest.mark.parametrize("cells", [524289, 1310721, 1572865, 1835009, 2097153])
def test_last_path_cells_arrive(cells):
    """Paths of `cells` cells in all along a corridor, the last one ending on the source."""
    import paper_2004_00540_amd as omap
    W, whole = 13000, cells // 12000 - 1
    rest = cells - whole * 12000            # two more paths make up the number
    tgt = np.array([[0, 11999]] * whole + [[0, rest // 2 - 1], [0, rest - rest // 2 - 1]], np.int32)
    m = workloads.Maze(np.zeros((1, W), np.uint8), np.zeros((1, 2), np.int32), tgt, "corridor")
    _, _, rl, ro, rc = oracle_solution(m, -1, closed_form=True)
    assert ro[-1] == cells
    with omap.Engine(1 << 28, max_slots=1) as eng:
        for _ in range(2):
            got = _solve(eng, m.occ, m.sources, tgt)
            assert np.array_equal(got.lengths, rl) and np.array_equal(got.offsets, ro) and np.array_equal(got.cells, rc)
