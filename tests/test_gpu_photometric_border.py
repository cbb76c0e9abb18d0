"""Visibility on the image border, which the projection decides: surface points
that project exactly on column 0 (seen) and exactly on column width-1 (not
seen) at many depths, where the quotient x / z is exact and only a quotient
rounded as a division gives it.  Expected view counts by float64 division."""
import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,seen", [(-1, 1.0), (1, 0.0)])
def test_points_on_the_border_columns(side, seen):
    import torch
    from paper_2111_13652_amd.gsdf import GsdfMap, PhotometricLoss, mean_color, voxel_order
    vs, T = 0.125, 4.0
    f, width, height = 100.0, 201, 21
    cam = synth.Camera(f, f, 100.0, 10.0, width, height, 0.3, 100.0)
    order = voxel_order()
    coords = np.array([[side * k, 0, k] for k in range(8, 73)])   # z = 1 .. 9, x = -z or z: columns 0 or 200
    z = coords[:, 2] * vs
    u = f * (coords[:, 0] * vs) / z + cam.cx
    assert (u == (0.0 if side < 0 else 200.0)).all()
    keys = np.unique(coords >> 3, axis=0).astype(np.int32)
    psi = np.zeros((len(keys), 512), np.float32)
    g = np.zeros((len(keys), 512, 3), np.float32)
    W = np.zeros((len(keys), 512), np.float32)
    index = {tuple(k): i for i, k in enumerate(keys)}
    for c in coords:
        l = c & 7
        W[index[tuple(c >> 3)], l[0] + 8 * l[1] + 64 * l[2]] = 1.0
    g[W > 0] = [0.0, 0.0, 1.0]
    G = GsdfMap(vs, T, 64)
    G.import_blocks(keys, psi, g, W)
    gk = G.keys()
    slot = {tuple(k): i for i, k in enumerate(gk)}
    params = G.export_params()
    D = dev(np.full((1, height, width), 5.0, np.float32))   # every z lies within the truncation of it
    rgb = dev(np.full((1, height, width, 3), 0.5, np.float32))
    T0 = dev(np.hstack([np.eye(3), np.zeros((3, 1))])[None])
    xi = dev(np.zeros((1, 6)))
    log(f"case: {len(coords)} points on column {int(u[0])}")
    _, cnt = mean_color(G, params, xi, D, rgb, cam, T0)
    cnt = cnt.cpu().numpy()[:, order]
    got = np.array([cnt[slot[tuple(c >> 3)], (c & 7)[0] + 8 * (c & 7)[1] + 64 * (c & 7)[2]] for c in coords])
    assert (got == seen).all(), f"{int((got != seen).sum())} of {len(got)} decided otherwise"
    loss = PhotometricLoss.apply(params, torch.zeros((len(gk), 512, 3), device="cuda"), xi, G, D, rgb, cam, T0, 1.0, 1.0)
    want = seen * len(coords) * 3 * 0.5 * 0.5 ** 2
    assert abs(float(loss.sum()) - want) <= 1e-6 * want
