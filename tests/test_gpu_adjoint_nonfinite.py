"""A keyframe whose pose is not finite (a NaN or infinite twist, a NaN in its
start pose) adds nothing to the gradients of the voxels that other keyframes
share with it: dparams, and the other keyframes' losses and pose gradients,
are the same bits as without it, with a frozen association and without one.
The map holds the block at the origin, which a NaN point rounds to."""
import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("freeze", [False, True])
@pytest.mark.parametrize("what", ["nan_xi", "inf_xi", "nan_T0"])
def test_a_nonfinite_keyframe_adds_nothing(what, freeze):
    import torch
    from paper_2111_13652_amd.gsdf import GsdfMap, KeyframeLoss, keyframe_loss
    rng = np.random.default_rng(3)
    width, height, K = 96, 72, 4
    cam = synth.Camera(80.0, 80.0, 47.5, 35.5, width, height, 0.3, 4.0)
    u, v = np.meshgrid(np.arange(width), np.arange(height))
    D = np.stack([0.8 / (1 - 0.2 * ((u - cam.cx) / cam.fx + 0.4 * (v - cam.cy) / cam.fy))
                  + 0.001 * rng.standard_normal(u.shape) for _ in range(K)]).astype(np.float32)
    eye = np.hstack([np.eye(3), np.array([[0.0], [0.0], [-0.8]])])   # the surface passes through the origin
    G = GsdfMap(0.02, 0.1, 2048)
    for k in range(2):
        G.fuse(dev(D[k]), cam, dev(eye))
    assert any(tuple(k) == (0, 0, 0) for k in G.keys())
    params = G.export_params()
    T0 = np.stack([synth.perturb_pose(eye, 3 + i, 0.5, 0.005) for i in range(K)])
    xi = 1e-3 * rng.standard_normal((K, 6))
    assoc = None
    if freeze:
        assoc = torch.empty((K, height, width, 3), dtype=torch.int32, device="cuda")
        keyframe_loss(G, params, dev(np.zeros((K, 6))), dev(D), cam, dev(T0), 0.01, assoc)
    if what == "nan_xi":
        xi[2, 4] = np.nan
    elif what == "inf_xi":
        xi[2, 0] = np.inf
    else:
        T0[2, 1, 3] = np.nan
    scale = np.array([1.0, 0.7, 0.5, 0.9], np.float32)
    got = []
    for rows in ([0, 1, 2, 3], [0, 1, 3]):
        P = params.clone().requires_grad_(True)
        X = dev(xi[rows]).requires_grad_(True)
        a = None if assoc is None else assoc[rows].contiguous()
        log(f"case: {what}, frozen {freeze}, keyframes {rows}")
        loss = KeyframeLoss.apply(P, X, G, dev(D[rows]), cam, dev(T0[rows]), 0.01, a, freeze)
        loss.backward(dev(scale[rows]).double())
        torch.cuda.synchronize()
        keep = [i for i, r in enumerate(rows) if r != 2]
        got.append((P.grad, X.grad[keep], loss.detach()[keep]))
    assert got[1][0].abs().max() > 0 and torch.isfinite(got[1][0]).all()
    for with_it, without in zip(*got):
        assert torch.equal(with_it, without)
