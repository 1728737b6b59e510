"""Batches of more mazes than one block of a start copies descriptors for (about
20), up to more than its blocks do at once, started again with other layers."""
import numpy as np
import pytest

import oracle
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 21, 37, 500, 26000])
def test_batch_of_many_small_mazes(n):
    import paper_2004_00540_amd as omap
    rng = np.random.default_rng(n)
    kinds = []
    for _ in range(16):
        occ = (rng.random((int(rng.integers(2, 20)), int(rng.integers(2, 24)))) < 0.3).astype(np.uint8)
        free = np.argwhere(occ == 0).astype(np.int32)
        src, tgt = free[:1], free[rng.integers(0, len(free), 2)]
        by_layers = {}
        for L in (-1, 3):
            d, ecc = oracle.bfs(occ, src)
            A = oracle.activity_from_bfs(d, ecc if L < 0 else L)
            by_layers[L] = (ecc if L < 0 else L, int((A > 0).sum()), *oracle.walk(A, src, tgt))
        kinds.append(((to_dev(occ), src, tgt), by_layers))
    pick = rng.integers(0, len(kinds), n)
    with omap.Batch([kinds[k][0] for k in pick]) as b:
        for L in (-1, 3, -1):
            infos = b.propagate([L] * n)
            refs = [kinds[k][1][L] for k in pick]
            assert [(i["layers"], i["reached_cells"]) for i in infos] == [r[:2] for r in refs]
            ln, off, cells = (t.cpu().numpy() for t in b.paths())
            assert np.array_equal(ln, np.concatenate([r[2] for r in refs]))
            assert np.array_equal(off, np.concatenate([[0], np.cumsum(np.where(ln >= 0, ln + 1, 0))]))
            assert np.array_equal(cells, np.concatenate([r[4] for r in refs]))
