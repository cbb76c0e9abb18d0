"""A keyframe's Gauss-Newton step is the same bits alone and in any batch: its
pixels are grouped by its own size, not by how many keyframes there are."""
import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests import scenes
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["fp32", "fp16"])
@pytest.mark.parametrize("K", [2, 110, 257])
def test_step_is_the_same_bits_in_any_batch(storage, K):
    from paper_2111_13652_amd.gsdf import GsdfMap
    cam = scenes.SMALL_CAM
    sc, T0 = scenes.box_room_scene(), scenes.box_room_pose()
    G = GsdfMap(0.02, 0.1, 4096, storage=storage)
    poses, depth = [], []
    for k in range(2):
        T = synth.perturb_pose(T0, 100 + k, 1.0, 0.01)
        d = synth.to_depth_image(synth.render_depth(sc, cam, T), cam).astype(np.float32)
        G.fuse(dev(d), cam, dev(T))
        poses.append(synth.perturb_pose(T, 7 + k, 0.5, 0.005))
        depth.append(d)
    rep = (K + 1) // 2
    P = dev(np.concatenate([np.stack(poses)] * rep)[:K].copy())
    G.gn_step_keyframes(dev(np.concatenate([np.stack(depth)] * rep)[:K]), cam, P)
    P = P.cpu().numpy()
    log(f"case: {K} keyframes, {storage}")
    for k in range(2):
        one = dev(poses[k][None].copy())
        G.gn_step_keyframes(dev(depth[k][None]), cam, one)
        assert all(np.array_equal(P[i], one.cpu().numpy()[0]) for i in range(k, K, 2))
    assert G.status_flags() == []
