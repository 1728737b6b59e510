"""Copy-out of the activity map: widths around a lane's four columns and a wave's
256, heights around a wave's four rows and a block's sixteen, destinations with
odd pitches and offsets, and nothing written outside the map."""
import numpy as np
import pytest

import workloads
from gpu_helpers import oracle_solution, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1), (3, 4), (4, 5), (5, 7), (15, 255), (16, 256), (17, 257), (33, 1021)])
@pytest.mark.parametrize("pitch,offset", [(0, 0), (1, 0), (3, 1), (64, 3)])
def test_activity_copy(shape, pitch, offset):
    import torch
    import paper_2004_00540_amd as omap
    H, W = shape
    m = workloads.random_maze(H, W, 0.2, 1, 2, 5100 + H + W)
    flat = torch.full((offset + H * (W + pitch) + 8,), -9, dtype=torch.int32, device="cuda")
    view = flat[offset:offset + H * (W + pitch)].view(H, W + pitch)
    A = oracle_solution(m, -1)[0]
    for schedule in (0, 1):                     # (1 with 8 layers: the integer sweep's buffers)
        flat.fill_(-9)
        with omap.Plan(to_dev(m.occ), m.sources, m.targets, schedule=schedule,
                       temporal_depth=8 if schedule else 0) as plan:
            plan.propagate()
            plan.activity(out=view)
        got = flat.cpu().numpy()
        inside = got[offset:offset + H * (W + pitch)].reshape(H, W + pitch)
        assert np.array_equal(inside[:, :W], A)
        assert (inside[:, W:] == -9).all() and (got[:offset] == -9).all() and (got[offset + H * (W + pitch):] == -9).all()
