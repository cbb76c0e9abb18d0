"""The batched Gauss-Newton step where its work-groups per keyframe change:
just below, at and above the number that fills the chip (a 160x120 keyframe
takes up to five of them), against the same keyframes one by one, which group
their pixels by five (bar 1e-7 rad / 1e-7 m, as for the regrouped float32
sums of the step against tracking)."""
import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests import scenes
from tests.gpu_helpers import dev, log, pose_diff

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["fp32", "bf16"])
@pytest.mark.parametrize("K", [102, 103, 230, 600])
def test_step_does_not_depend_on_the_batch(storage, K):
    import torch
    from paper_2111_13652_amd.gsdf import GsdfMap
    cam = synth.Camera(131.0, 131.0, 79.5, 59.5, 160, 120, 0.4, 4.0)
    sc, T0 = scenes.box_room_scene(), scenes.box_room_pose()
    G = GsdfMap(0.02, 0.1, 4096, storage=storage)
    poses, depth = [], []
    for k in range(4):
        T = synth.perturb_pose(T0, 100 + k, 1.0, 0.01)
        d = synth.to_depth_image(synth.render_depth(sc, cam, T), cam).astype(np.float32)
        G.fuse(dev(d), cam, dev(T))
        poses.append(synth.perturb_pose(T, 7 + k, 0.5, 0.005))
        depth.append(d)
    poses, depth = np.stack(poses), np.stack(depth)
    one = []
    for k in range(4):
        P = dev(poses[k:k + 1].copy())
        G.gn_step_keyframes(dev(depth[k:k + 1]), cam, P)
        one.append(P.cpu().numpy()[0])
    rep = (K + 3) // 4
    P = dev(np.concatenate([poses] * rep)[:K].copy())
    G.gn_step_keyframes(dev(np.concatenate([depth] * rep)[:K]), cam, P)
    assert G.status_flags() == []
    P = P.cpu().numpy()
    worst = max(max(pose_diff(P[i], one[i % 4])) for i in range(K))
    log(f"case: {K} keyframes, {storage}: worst difference {worst:.2e}")
    assert worst < 1e-7
    for i in range(4, K):
        assert np.array_equal(P[i], P[i % 4])
    if storage == "bf16":   # its grouping does not change with the batch
        assert all(np.array_equal(P[i], one[i]) for i in range(4))
