"""Tracking's bounded waits in the 16-bit form, whose sums have a barrier of
their own: with every wait bounded to one poll each work-group leaves as a
whole, the frame is reported as given up, and the next call on the same map
and scratch, with the default bounds, has the bits of an undisturbed one."""
import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests import scenes
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["bf16", "fp16"])
@pytest.mark.parametrize("width,height,levels,iters", [(160, 120, 1, (6,)), (640, 480, 3, (4, 5, 10))])
def test_sixteen_bit_tracking_gives_up_and_recovers(storage, width, height, levels, iters):
    import torch
    from paper_2111_13652_amd.gsdf import GsdfMap
    s = width / 160.0
    cam = synth.Camera(131.0 * s, 131.0 * s, (width - 1) / 2.0, (height - 1) / 2.0, width, height, 0.4, 4.0)
    sc, T0 = scenes.box_room_scene(), scenes.box_room_pose()
    G = GsdfMap(0.02, 0.1, 4096, storage=storage)
    d0 = synth.to_depth_image(synth.render_depth(sc, cam, T0), cam).astype(np.float32)
    G.fuse(dev(d0), cam, dev(T0))
    T1 = synth.perturb_pose(T0, 11, 0.5, 0.005)
    D = dev(synth.to_depth_image(synth.render_depth(sc, cam, T1), cam).astype(np.float32))
    ref = dev(T0.copy())
    G.track(D, cam, ref, levels=levels, iters=iters)
    torch.cuda.synchronize()
    assert G.status_flags() == []
    log(f"case: {storage} {width}x{height}, every wait bounded to one poll")
    out = dev(T0.copy())
    G.track(D, cam, out, levels=levels, iters=iters, max_polls=1)
    torch.cuda.synchronize()        # every work-group exited
    assert "gave_up" in G.status_flags()
    G.status.zero_()
    P = dev(T0.copy())
    G.track(D, cam, P, levels=levels, iters=iters)
    torch.cuda.synchronize()
    assert G.status_flags() == []
    assert torch.equal(P, ref)
