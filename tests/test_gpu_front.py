"""The bit-packed front propagation (the default of plans, batches and engines)
at the edges of its tiles (64 x 64 cells), words (32 cells), steps (16 layers)
and rounds (64 layers): maps, layer and reached-cell counts and paths against
the oracle's literal layers, bit for bit."""
import numpy as np
import pytest

import workloads
from gpu_helpers import assert_same, oracle_solution, run_plan, to_dev

pytestmark = pytest.mark.gpu

LAYERS = (-1, 0, 1, 15, 16, 17, 47, 48, 49, 63, 64, 65, 127, 128, 129, 193)


@pytest.mark.parametrize("shape", [(1, 1), (1, 65), (65, 1), (2, 33), (63, 64), (64, 63), (64, 65), (65, 31),
                                   (129, 127), (128, 193), (191, 257), (40, 700), (700, 40)])
@pytest.mark.parametrize("density", [0.0, 0.3])
def test_front_edges(shape, density):
    H, W = shape
    m = workloads.random_maze(H, W, density, 2, 12, 4100 + 3 * H + W)
    m.sources = np.concatenate([m.sources, m.sources[:1]])      # a source listed twice counts once
    for L in LAYERS:
        print(f"front {shape} density={density} L={L}", flush=True)
        assert_same(m, run_plan(m, L), oracle_solution(m, L), f"front {shape} density={density} L={L}")


@pytest.mark.parametrize("shape", [(1, 1), (64, 64), (65, 129), (191, 257), (40, 700)])
def test_front_dense_schedule(shape):
    """Every tile in every round until the maze stops changing."""
    H, W = shape
    m = workloads.random_maze(H, W, 0.3, 2, 12, 4300 + 3 * H + W)
    for L in LAYERS:
        assert_same(m, run_plan(m, L, schedule=2), oracle_solution(m, L), f"front dense {shape} L={L}")


@pytest.mark.parametrize("corner", [(0, 0), (63, 63), (64, 64), (127, 64), (128, 129)])
def test_front_straight_into_every_neighbour(corner):
    """One source at a tile's corner on an empty map: the front enters the
    neighbour tiles in the layers just before and after a round's last."""
    occ = np.zeros((200, 200), np.uint8)
    tgt = np.array([[0, 0], [199, 199], [0, 199], [199, 0]], np.int32)
    m = workloads.Maze(occ, np.array([corner], np.int32), tgt, f"corner{corner}")
    for L in (-1, 62, 63, 64, 65, 66):
        assert_same(m, run_plan(m, L), oracle_solution(m, L), f"corner {corner} L={L}")


@pytest.mark.parametrize("schedule", [0, 2])
def test_front_batch_of_mixed_layer_counts_and_reuse(schedule):
    """Mazes that end in different rounds, propagated again with other counts
    (the planes of a tile last visited in an odd round are cleared too)."""
    import paper_2004_00540_amd as omap
    ms = [workloads.random_maze(30 + 37 * i, 333 - 31 * i, 0.3, 1 + i % 3, 9, 4200 + i) for i in range(9)]
    with omap.Batch([(to_dev(m.occ), m.sources, m.targets) for m in ms], schedule=schedule) as b:
        for rep in range(3):
            layers = [(-1, 3 + 20 * i, 64, 128, 70 + i)[(i + rep) % 5] for i in range(len(ms))]
            infos = b.propagate(layers)
            for i, m in enumerate(ms):
                A, L, *_ = oracle_solution(m, layers[i])
                assert np.array_equal(b.activity(i).cpu().numpy(), A), (rep, i)
                assert (infos[i]["layers"], infos[i]["reached_cells"]) == (L, int((A > 0).sum())), (rep, i)


@pytest.mark.parametrize("joined", [False, True])
def test_front_in_some_words(joined):
    """Fronts in every subset of six neighbouring 32-column words: a wave
    advances the words that gain cells and those beside them."""
    import oracle
    import paper_2004_00540_amd as omap
    H, words, first = 150, 10, 2
    rng = np.random.default_rng(61)
    base = (rng.random((H, 32 * words)) < 0.35).astype(np.uint8)
    ms = []
    for subset in range(1, 64):
        occ = base.copy()
        src = []
        for w in range(words):
            c0, c1 = 32 * w, 32 * w + 31
            if not joined:
                occ[:, [c0, c1]] = 1               # a chamber per word
            if 0 <= w - first < 6 and subset >> (w - first) & 1:
                r, c = 40 + 10 * (w - first), c0 + (1, 16, 30)[w % 3]
                occ[r, c] = 0
                src.append((r, c))
        ms.append((occ, np.array(src, np.int32)))
    with omap.Batch([(to_dev(o), s, s[:1]) for o, s in ms]) as b:
        infos = b.propagate()
        for i, (o, s) in enumerate(ms):
            d, ecc = oracle.bfs(o, s)
            assert infos[i]["layers"] == ecc, i + 1
            assert np.array_equal(b.activity(i).cpu().numpy(), oracle.activity_from_bfs(d, ecc)), i + 1
