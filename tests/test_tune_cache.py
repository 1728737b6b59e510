"""The autotuner's saved choices: an entry is read back only by the kernels it
was timed with.  Needs no GPU: without a device the call ends at its first
allocation unless the file already answers it."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2004_00540_amd as omap

pytestmark = pytest.mark.skipif(torch.cuda.is_available(), reason="the occupancy pointer is not a device one")


def _tune_plan():
    src = np.zeros((1, 2), np.int32)
    desc = (omap.MazeDesc * 1)(omap.MazeDesc(16, 16, 0x1000, src.ctypes.data, 1, None, 0))
    res = omap.TuneResult()
    st = omap.lib().omap_tune(desc, 1, omap.USE_PLAN, ctypes.byref(res), None)
    return omap.STATUS[st], res.from_cache


@pytest.mark.parametrize("tag", ["", " kernels=0", " kernels=00000000"])
def test_entry_of_other_kernels_is_not_used(tmp_path, monkeypatch, tag):
    cache = tmp_path / "tune.txt"
    cache.write_text(f"unknown use0 n2^0 cells2^8{tag} = 1 12 1 12 0\n")
    monkeypatch.setenv("OMAP_TUNE_CACHE", str(cache))
    status, from_cache = _tune_plan()
    assert status != "OMAP_OK" and from_cache == 0
