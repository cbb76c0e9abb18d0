"""Tracking's sums on the levels that one XCD works, where a thread holds up to
two pixels.  On a lone sphere, whose rotations about its centre leave the
residuals unchanged, the damping amplifies the rounding of the sums, and the
observable part of the pose is the sphere's centre in the camera.  A thread's
values are added in float64 there, so fewer float32 roundings enter than in
float32 sums of four single pixels, with which this configuration's centre
came within 1e-7 m of the FP64 oracle's; the bar is ten times that."""
import numpy as np
import pytest

import oracle
from paper_2111_13652_amd import synth
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


def test_sphere_centre_on_a_small_level():
    from paper_2111_13652_amd.gsdf import GsdfMap
    cfg = synth.CONFIG_SPHERE
    cam = cfg["cam"]
    sc = synth.sphere_scene()
    T0 = np.hstack([np.eye(3), np.zeros((3, 1))])
    d0 = synth.to_depth_image(synth.render_depth(sc, cam, T0), cam)
    d1 = synth.to_depth_image(synth.render_depth(sc, cam, synth.perturb_pose(T0, 0, 2.0, 0.02)), cam)
    bounds = ([-4, -4, 5], [4, 4, 13])
    O = oracle.OracleMap(0.02, 0.10, bounds=bounds)
    G = GsdfMap(0.02, 0.10, 1024, bounds=bounds)
    O.allocate(d0, cam, T0)
    O.integrate(d0, cam, T0)
    G.allocate(dev(d0), cam, dev(T0))
    G.integrate(dev(d0), cam, dev(T0))
    To, _, _ = O.track(d1, cam, T0, 1, [10], 0.01)
    P = dev(T0.copy())
    G.track(dev(d1), cam, P, levels=1, iters=(10,), delta=0.01)
    Tg = P.cpu().numpy()
    centre = lambda T: T[:, :3].T @ (np.array([0.0, 0.0, 1.5]) - T[:, 3])
    err = float(np.linalg.norm(centre(Tg) - centre(To)))
    log(f"case: {cam.width}x{cam.height}, sphere centre GPU-oracle {err:.2e} m")
    assert err < 1e-6
