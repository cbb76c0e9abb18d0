"""Allocation alone, called for many frames before any is integrated: the
per-block pixel counts that size fusion's pieces add up over the calls (past
2^31 pixels for the block in front of the camera here) and must stay a mark
that the block is touched.  The map is the same bits as after one call."""
import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("calls", [600, 1100])
def test_allocation_many_times_before_integration(calls):
    import torch
    from paper_2111_13652_amd.gsdf import GsdfMap
    size = 2048   # four million pixels a call
    cam = synth.Camera(6000.0, 6000.0, (size - 1) / 2, (size - 1) / 2, size, size, 0.3, 4.0)
    D = torch.full((size, size), 1.0, dtype=torch.float32, device="cuda")
    pose = dev(np.hstack([np.eye(3), np.array([[0.4], [0.4], [0.0]])]))
    maps = []
    for n in (1, calls):
        m = GsdfMap(0.1, 0.3, 64)
        for _ in range(n):
            m.allocate(D, cam, pose)
        m.integrate(D, cam, pose)
        torch.cuda.synchronize()
        assert m.status_flags() == []
        keys = m.keys()
        o = np.lexsort(keys.T[::-1])
        maps.append([keys[o]] + [x[o] for x in m.voxels(len(keys))])
    log(f"case: {calls} calls, {len(maps[0][0])} blocks, weight {maps[0][3].sum():.0f} and {maps[1][3].sum():.0f}")
    assert maps[0][3].sum() > 0
    for a, b in zip(*maps):
        assert np.array_equal(a, b)
