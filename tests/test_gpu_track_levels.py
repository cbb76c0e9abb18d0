"""Tracking where its levels change hands: levels up to 24576 pixels are worked
by one XCD, larger ones by the whole grid, whose other work-groups take the
pose at the boundary.  Sizes at, just below and just above the limit, alone
and as the coarse level of a pyramid, and an image of fewer pixels than
work-group lanes, against the oracle; through device scope the same bits."""
import numpy as np
import pytest

import oracle
from paper_2111_13652_amd import synth
from tests import scenes
from tests.gpu_helpers import dev, log, pose_diff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height,levels,iters", [
    (24, 16, 1, (6,)),            # one pixel or none to a lane
    (192, 128, 1, (6,)),          # 24576 pixels
    (193, 128, 1, (6,)),          # one column more: the whole grid
    (384, 256, 2, (3, 4)),        # from one XCD to the grid
    (386, 256, 2, (3, 4)),        # the grid on both levels
    (384, 256, 4, (2, 0, 3, 3)),  # a level left out at the boundary
])
def test_levels_at_the_one_xcd_limit(width, height, levels, iters):
    import torch
    from paper_2111_13652_amd.gsdf import GsdfMap
    s = width / 160.0
    cam = synth.Camera(131.0 * s, 131.0 * s, (width - 1) / 2.0, (height - 1) / 2.0, width, height, 0.4, 4.0)
    sc, T0 = scenes.box_room_scene(), scenes.box_room_pose()
    O = oracle.OracleMap(0.02, 0.1)
    big = synth.Camera(131.0, 131.0, 79.5, 59.5, 160, 120, 0.4, 4.0)
    for k in range(3):
        Tk = synth.perturb_pose(T0, 100 + k, 1.0, 0.01)
        d = synth.to_depth_image(synth.render_depth(sc, big, Tk), big)
        O.allocate(d, big, Tk)
        O.integrate(d, big, Tk)
    T1 = synth.perturb_pose(T0, 11, 0.5, 0.005)
    depth = synth.to_depth_image(synth.render_depth(sc, cam, T1), cam).astype(np.float32)
    keys = O.keys()
    psi, g, W, _ = O.voxels(keys)
    G = GsdfMap(0.02, 0.1, 4096)
    G.import_blocks(keys, psi, g, W)
    log(f"case: {width}x{height}, {levels} levels, iterations {iters}")
    To, so, failed = O.track(depth, cam, T0, levels, list(iters), 0.01)
    out = []
    for scope in (False, True):
        P = dev(T0.copy())
        stats = torch.zeros(2 * sum(iters), dtype=torch.float32, device="cuda")
        G.track(dev(depth), cam, P, levels=levels, iters=iters, delta=0.01, stats=stats, device_scope=scope)
        out.append(P)
    assert G.status_flags() == []
    assert torch.equal(out[0], out[1])
    dr, dt = pose_diff(out[0].cpu().numpy(), To)
    log(f"  GPU vs oracle: {dr:.2e} rad, {dt:.2e} m")
    assert dr < 1e-5 and dt < 1e-5
    sg = stats.cpu().numpy().reshape(-1, 2)
    np.testing.assert_allclose(sg[:, 1], so[:, 1], rtol=1e-4)
    np.testing.assert_allclose(sg[:, 0], so[:, 0], rtol=1e-3)
