"""The photometric kernels where their layout can go wrong: blocks with few,
with more than 64, more than 128 and all 512 of their voxels on the surface,
and keyframe counts around the batches that the waves take together, against
the FP64 oracle with the bars of the photometric parity test."""
import numpy as np
import pytest

import oracle
from paper_2111_13652_amd import synth
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fill,K", [(0.05, 1), (0.2, 5), (0.4, 8), (1.0, 9), (1.0, 17)])
def test_dense_blocks_and_keyframe_batches(fill, K):
    import torch
    from paper_2111_13652_amd.gsdf import GsdfMap, MeanColor, PhotometricLoss, mean_color, voxel_order
    rng = np.random.default_rng(int(100 * fill) + K)
    vs, T = 0.01, 0.05
    cam = synth.Camera(80.0, 80.0, 47.5, 35.5, 96, 72, 0.3, 4.0)
    keys = np.array([[x, y, z] for z in (12, 13) for y in (-1, 0) for x in (-1, 0, 1)], np.int32)
    n = len(keys)
    g = np.array([0.0, 0.0, 1.0]) + 0.3 * rng.standard_normal((n, 512, 3))
    g = (5.0 * g / np.linalg.norm(g, axis=-1, keepdims=True)).astype(np.float32)
    psi = np.where(rng.random((n, 512)) < fill, rng.uniform(-0.004, 0.004, (n, 512)), 0.04).astype(np.float32)
    W = np.where(rng.random((n, 512)) < 0.95, 5.0, 0.0).astype(np.float32)
    g[W == 0] = 0.0
    psi[W == 0] = 0.0
    G = GsdfMap(vs, T, 64)
    G.import_blocks(keys, psi, g, W)
    order = voxel_order()
    gk = G.keys()
    params = G.export_params(n)
    p = params.cpu().numpy()[:, order, :]
    Wl = G.weight[: n * 512].view(n, 512).cpu().numpy()[:, order]
    O = oracle.OracleMap(vs, T)
    O.set_voxels(gk, p[..., 0].astype(np.float64), p[..., 1:].astype(np.float64), Wl.astype(np.float64))
    D = (1.02 + 0.01 * rng.standard_normal((K, 72, 96))).astype(np.float32)
    I = rng.uniform(0.2, 0.8, (K, 72, 96, 3)).astype(np.float32)
    eye = np.hstack([np.eye(3), np.zeros((3, 1))])
    T0 = np.stack([synth.perturb_pose(eye, 7 + i, 1.0, 0.02) for i in range(K)])
    xi = 1e-3 * rng.standard_normal((K, 6))
    args = (dev(D), dev(I), cam, dev(T0))

    col_o, cnt_o = O.mean_color(D.astype(np.float64), I.astype(np.float64), cam, T0, xi, gk)
    col, cnt = mean_color(G, params, dev(xi), *args)
    log(f"case: fill {fill}, {K} keyframes: {int((cnt_o > 0).sum(axis=1).max())} voxels of a block seen")
    np.testing.assert_array_equal(cnt.cpu().numpy()[:, order], cnt_o)
    np.testing.assert_allclose(col.cpu().numpy()[:, order], col_o, atol=2e-6)

    rho = np.clip(col_o + 0.05 * rng.standard_normal(col_o.shape), 0, 1).astype(np.float32)
    delta, lam = 0.05, 0.8
    L_o, dpsi_o, dcol_o, dxi_o, _ = O.photo_loss_grad(D.astype(np.float64), I.astype(np.float64), cam, T0, xi,
                                                      rho.astype(np.float64), delta, lam, gk)
    P = params.clone().requires_grad_(True)
    R = torch.empty_like(dev(rho))
    R[:, torch.as_tensor(order.astype(np.int64)).cuda()] = dev(rho)
    R.requires_grad_(True)
    X = dev(xi).requires_grad_(True)
    L = PhotometricLoss.apply(P, R, X, G, *args, delta, lam)
    L.sum().backward()
    np.testing.assert_allclose(L.detach().cpu().numpy(), L_o, rtol=1e-5)
    assert (np.abs(X.grad.cpu().numpy() - dxi_o).max(axis=1) < 1e-4 * np.abs(dxi_o).max(axis=1)).all()
    for gpu, orc in ((P.grad.cpu().numpy()[:, order, 0], dpsi_o), (R.grad.cpu().numpy()[:, order], dcol_o)):
        assert np.abs(orc).max() > 0
        assert (np.abs(gpu - orc) <= 1e-4 * np.abs(orc) + 1e-6 * np.abs(orc).max()).all()

    # the mean colour's adjoint: linear in the upstream gradient, so two
    # halves of it add up to the whole
    up = torch.randn(col.shape, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    out = []
    for w in (up, torch.where(up > 0, up, 0.0), torch.where(up > 0, 0.0, up)):
        P, X = params.clone().requires_grad_(True), dev(xi).requires_grad_(True)
        MeanColor.apply(P, X, G, *args)[0].backward(w)
        out.append((P.grad, X.grad))
    for whole, a, b in zip(*out):
        assert whole.abs().max() > 0
        assert (whole - (a + b)).abs().max() <= 2e-5 * (a.abs() + b.abs()).max()
