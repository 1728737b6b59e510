"""Offsets and paths of more targets than one block scans (1,024), at the edges of
the scan's blocks (256 targets) and of the blocks that one block scans (256 of
them), for each kind of walk and for an engine's retirement."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu

COUNTS = (1024, 1025, 1280, 4095, 4096, 4097, 4352, 4353, 65536, 65537)


def _problem(n):
    """A maze with unreached targets, and n targets drawn from its free cells."""
    m = workloads.random_maze(60, 70, 0.42, 2, 4, 77)
    free = np.argwhere(m.occ == 0).astype(np.int32)
    pick = np.random.default_rng(n).integers(0, len(free), n)
    d, ecc = oracle.bfs(m.occ, m.sources)
    return m, oracle.activity_from_bfs(d, ecc), free, pick


def _expand(ref, pick):
    """The results of targets `pick` from those of every free cell."""
    ln, off, cells = ref
    n_cells = np.maximum(ln + 1, 0)[pick]
    out = np.concatenate([[0], np.cumsum(n_cells)]).astype(np.int64)
    at = np.repeat(off[:-1][pick] - out[:-1], n_cells) + np.arange(out[-1])
    return ln[pick], out, cells[at]


@pytest.mark.parametrize("n", COUNTS)
def test_many_targets(n):
    import paper_2004_00540_amd as omap
    m, A, free, pick = _problem(n)
    targets = free[pick]
    with omap.Plan(to_dev(m.occ), m.sources, targets) as plan:
        plan.propagate()
        for mode in (None, "euclidean"):
            walk = oracle.walk_euclidean if mode else oracle.walk
            ref = _expand(walk(A, m.sources, free), pick)
            assert (ref[0] < 0).any() and (ref[0] >= 0).any()
            for g, r in zip(plan.paths(mode), ref):
                assert np.array_equal(g.cpu().numpy(), r), (n, mode)
        got = plan.paths("random", 5)
        assert np.array_equal(got[1].cpu().numpy(), _expand(oracle.walk(A, m.sources, free), pick)[1])
    with omap.Engine(1 << 28) as e:
        qid = e.submit(m.occ, m.sources, targets)
        for _ in range(200):
            e.step()
            if e.poll(qid) in (omap.QUERY_DONE, omap.QUERY_FAILED):
                break
        res = e.fetch(qid)
    ref = _expand(oracle.walk(A, m.sources, free), pick)
    for g, r in zip((res.lengths, res.offsets, res.cells), ref):
        assert np.array_equal(g, r), n


@pytest.mark.parametrize("layers", [-1, 0, 40, 1 << 24])
def test_euclidean_walked_once_or_twice(layers):
    """The walk writes its points as it counts them where the layers are known and
    few enough, and walks twice otherwise: plans and a batch, layers known or not."""
    import paper_2004_00540_amd as omap
    m, _, free, pick = _problem(300)
    d, ecc = oracle.bfs(m.occ, m.sources)
    ref = _expand(oracle.walk_euclidean(oracle.activity_from_bfs(d, ecc if layers < 0 else layers), m.sources, free), pick)
    occ = to_dev(m.occ)
    for sync in (True, False):
        with omap.Plan(occ, m.sources, free[pick]) as plan:
            plan.propagate(layers, sync=sync)
            for _ in range(2):
                for g, r in zip(plan.paths("euclidean"), ref):
                    assert np.array_equal(g.cpu().numpy(), r), (layers, sync)
        with omap.Batch([(occ, m.sources, free[pick]), (occ, m.sources, free[pick][:0])]) as b:
            b.propagate([layers, layers], sync=sync)
            for g, r in zip(b.paths("euclidean")[:3], ref):
                assert np.array_equal(g.cpu().numpy(), r), (layers, sync)
