"""A program that uses the package before it has imported torch itself."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

PROGRAM = """
import numpy as np
import paper_2004_00540_amd as omap
assert omap.version() and omap.resolve_options()
with omap.Engine(1 << 20, max_slots=1) as eng:
    q = eng.submit(np.zeros((9, 9), np.uint8), [(4, 4)], [(0, 0)])
    while eng.poll(q) != omap.QUERY_DONE:
        eng.step()
    assert eng.fetch(q).lengths[0] == 4
import torch
with omap.Plan(torch.zeros((9, 9), dtype=torch.uint8, device="cuda"), [(4, 4)]) as plan:
    assert plan.propagate()["layers"] == 4
print("done")
"""


def test_library_before_torch():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", PROGRAM], cwd=root, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip() == "done", r.stderr[-2000:]
