"""Random-tie and Euclidean walks on both sides of the number of targets from which
they take a lane per target instead of a wave, against the oracle: plans and
batches, unreached targets, fixed and run-time layer counts."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode,n", [("random", 65536), ("random", 65537), ("euclidean", 20480), ("euclidean", 20481),
                                    ("euclidean", 131072)])
@pytest.mark.parametrize("layers", [-1, 25])
def test_lane_and_wave_walks(mode, n, layers):
    import paper_2004_00540_amd as omap
    a = workloads.random_maze(67, 130, 0.38, 2, 4, 31)
    b = workloads.random_maze(40, 61, 0.3, 3, 4, 32)
    rng = np.random.default_rng(n)
    refs, mazes = [], []
    for m, k in ((a, n - 100), (b, 100)):
        d, ecc = oracle.bfs(m.occ, m.sources)
        A = oracle.activity_from_bfs(d, ecc if layers < 0 else layers)
        targets = rng.integers(0, (m.H, m.W), (k, 2)).astype(np.int32)   # obstacles and unreached cells too
        refs.append(oracle.walk_random(A, m.sources, targets, 99) if mode == "random"
                    else oracle.walk_euclidean(A, m.sources, targets))
        mazes.append((to_dev(m.occ), m.sources, targets))
    assert all((r[0] < 0).any() and (r[0] > 0).any() for r in refs)
    want = (np.concatenate([refs[0][0], refs[1][0]]), np.concatenate([refs[0][1], refs[1][1][1:] + refs[0][1][-1]]),
            np.concatenate([refs[0][2], refs[1][2]]))
    with omap.Batch(mazes) as batch:
        batch.propagate([layers, layers])
        for g, r in zip(batch.paths(mode, 99), want):
            assert np.array_equal(g.cpu().numpy(), r), "batch"
    occ, src, tgt = mazes[0]
    pad = np.concatenate([tgt, tgt[:100]])           # n targets on one plan
    d, ecc = oracle.bfs(a.occ, a.sources)
    A = oracle.activity_from_bfs(d, ecc if layers < 0 else layers)
    ref = oracle.walk_random(A, src, pad, 99) if mode == "random" else oracle.walk_euclidean(A, src, pad)
    with omap.Plan(occ, src, pad) as plan:
        plan.propagate(layers)
        ln, off, cells, at = (t.cpu().numpy() for t in plan.paths(mode, 99, source_index=True))
    for g, r in zip((ln, off, cells), ref):
        assert np.array_equal(g, r), "plan"
    lin = src[:, 0].astype(np.int64) * a.W + src[:, 1]
    assert np.array_equal(at >= 0, ln >= 0) and np.array_equal(lin[at[ln >= 0]], cells[off[1:][ln >= 0] - 1])


def test_many_euclidean_paths_take_no_more_than_their_walks():
    """Asked for and taken, Euclidean paths are walked three times and random-tie
    paths once, move by move at a similar cost, beside scans that both have: so no
    more than three times as long (measured 1.8; with a wave per target 5.0)."""
    import torch
    import paper_2004_00540_amd as omap
    H = 1000
    targets = np.random.default_rng(3).integers(0, H, (1 << 19, 2)).astype(np.int32)
    with omap.Plan(torch.zeros((H, H), dtype=torch.uint8, device="cuda"), [(100, 100), (100, 900), (900, 100), (900, 900)],
                   targets) as plan:
        plan.propagate()

        def median_ms(mode):
            plan.paths(mode)
            out = []
            for _ in range(5):
                a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                a.record()
                plan.paths(mode)
                b.record()
                b.synchronize()
                out.append(a.elapsed_time(b))
            return sorted(out)[2]

        random, euclid = median_ms("random"), median_ms("euclidean")
    assert euclid <= 3 * random, (euclid, random)
