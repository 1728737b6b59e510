"""omap_plan_load reuses the plan's device buffers: a reload neither allocates nor
frees, so it does not wait for work on other streams."""
import numpy as np
import pytest

import oracle
import workloads
from gpu_helpers import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_sources", [1, 700])
def test_reload_does_not_wait_for_other_streams(n_sources):
    import torch
    import paper_2004_00540_amd as omap
    mazes = [workloads.random_maze(90, 130, 0.2, n_sources, 5, seed) for seed in (11, 12)]
    occ = [to_dev(m.occ) for m in mazes]
    own = torch.cuda.Stream()
    torch.cuda.synchronize()
    with omap.Plan(occ[0], mazes[0].sources, mazes[0].targets, stream=own) as plan:
        plan.propagate()
        plan.load(occ[1], mazes[1].sources, mazes[1].targets)   # (first use of every path)
        ran_on = []
        for _ in range(6):     # (a stream may share the plan's hardware queue, not all of them)
            with torch.cuda.stream(torch.cuda.Stream()):
                torch.cuda._sleep(50_000_000)     # one thread, tens of milliseconds
                done = torch.cuda.Event()
                done.record()
            plan.load(occ[0], mazes[0].sources, mazes[0].targets)
            ran_on.append(not done.query())
            torch.cuda.synchronize()
        assert any(ran_on)
        for k in (0, 1, 0):
            m = mazes[k]
            plan.load(occ[k], m.sources, m.targets)
            A, L = oracle.layers(m.occ, m.sources, -1)
            assert plan.propagate()["layers"] == L
            torch.cuda.synchronize()
            with torch.cuda.stream(own):
                act = plan.activity()
            own.synchronize()
            assert np.array_equal(act.cpu().numpy(), A)
