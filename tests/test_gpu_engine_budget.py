"""The engine's memory limit of a query: two int32 activity maps, the masks (bit
planes too under the bit-sliced schedule) at the maze's own height, the occupancy
and path scratch.  A budget of exactly that takes the query and solves it, also for
mazes lower than the kernels' layout granularity."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import workloads
from gpu_helpers import oracle_solution

pytestmark = pytest.mark.gpu


def _limit(H, W, n_targets, planes):
    pitch = (W + 63) // 64 * 64
    return (2 * 4 * pitch * H + planes * pitch // 8 * H + 4096 + H * W + 256 + n_targets * 64 +
            n_targets * 4 * (H + W) + 4096)


BITS, DENSE = {}, {"schedule": 2}


@pytest.mark.parametrize("H,W,opts,planes", [(1, 120000, BITS, 3), (2, 150001, BITS, 3), (15, 30000, BITS, 3),
                                             (16, 30000, BITS, 3), (17, 30001, BITS, 3), (300, 1000, BITS, 3),
                                             (15, 15000, DENSE, 1), (17, 14001, DENSE, 1), (300, 1000, DENSE, 1)])
def test_budget_of_exactly_the_limit_takes_the_query(H, W, opts, planes):
    import paper_2004_00540_amd as omap
    m = workloads.random_maze(H, W, 0.1 if H > 2 else 0.0, 2, 3, seed=H + W)
    budget = _limit(H, W, len(m.targets), planes)
    assert budget >= 1 << 20
    with omap.Engine(budget, max_slots=2, **opts) as eng:
        qid = eng.submit(m.occ, m.sources, m.targets)
        for _ in range(20000):
            eng.step(rounds=4)
            if eng.poll(qid) in (omap.QUERY_DONE, omap.QUERY_FAILED):
                break
        assert eng.poll(qid) == omap.QUERY_DONE
        got = eng.fetch(qid)
    A, L, rl, ro, rc = oracle_solution(m, -1, closed_form=True)
    assert got.info["layers"] == L and got.info["reached_cells"] == int((A > 0).sum())
    assert np.array_equal(got.lengths, rl) and np.array_equal(got.offsets, ro) and np.array_equal(got.cells, rc)
    with omap.Engine((budget - 256) // 256 * 256, max_slots=2, **opts) as eng:
        with pytest.raises(omap.OmapError) as e:
            eng.submit(m.occ, m.sources, m.targets)
        assert e.value.name == "OMAP_ERR_OUT_OF_MEMORY"
