"""Which kernel the benchmarks charge a propagation to: the helper against the
interface's words (no GPU) and against what ran (a round of the bit-packed kernel
is 64 layers, which no integer sweep applies)."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library)

import bench_forms
import paper_2004_00540_amd as omap

PLAN = [({}, True), ({"schedule": 1}, True), ({"schedule": 2}, True), ({"schedule": 3}, True),
        ({"temporal_depth": 16}, True), ({"lane_columns": 1}, True), ({"tile_rows": 16}, True),
        ({"schedule": 3, "temporal_depth": 8, "tile_rows": 32}, True),
        ({"schedule": 2, "temporal_depth": 16, "tile_rows": 256, "lane_columns": 4}, True),
        ({"temporal_depth": 12}, False), ({"lane_columns": 2}, False), ({"tile_rows": 32}, False),
        ({"schedule": 2, "tile_rows": 128}, False), ({"schedule": 2, "lane_columns": 2}, False)]
MANY = [({}, True), ({"schedule": 1}, False), ({"schedule": 2}, True), ({"schedule": 3}, True),
        ({"temporal_depth": 8}, True), ({"temporal_depth": 16, "tile_rows": 64}, True), ({"temporal_depth": 12}, False),
        ({"lane_columns": 1}, False), ({"schedule": 1, "temporal_depth": 16, "tile_rows": 16, "lane_columns": 1}, False),
        ({"schedule": 2, "temporal_depth": 8}, False)]
CASES = [(o, False, w) for o, w in PLAN] + [(o, True, w) for o, w in MANY]


@pytest.mark.parametrize("options,many,front", CASES)
def test_kernel_of_options(options, many, front):
    assert bench_forms.runs_front(options, many) is front


def test_work_of_a_propagation():
    work = bench_forms.propagation_work(True, 10 ** 9, 100, 5000)
    assert work["bytes"] == 100 * 64 * 64 * 3 / 8 + 4 * 5000 and work["ops_per_cell_update"] == 6 / 32
    assert bench_forms.propagation_work(False, 1000, 100, 5000)["bytes"] == 8125


@pytest.mark.gpu
@pytest.mark.parametrize("options,many,front", CASES)
def test_kernel_that_ran(options, many, front):
    import torch
    occ = torch.zeros((200, 300), dtype=torch.uint8, device="cuda")
    if many:
        with omap.Batch([(occ, [(0, 0)], None)], **options) as b:
            info = b.propagate()[0]
    else:
        with omap.Plan(occ, [(0, 0)], **options) as plan:
            info = plan.propagate()
    assert info["layers"] == 299
    assert (info["sweeps_executed"] == 64 * info["rounds"]) is bool(front), info
    assert np.int64(info["rounds"]) > 0
