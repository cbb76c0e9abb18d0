"""The adjoint's gather in parts: a block that many pixels see is gathered by
several work-groups, whose fixed-point sums give the same bits as one
work-group's, with one tile of the block scan and with several, with and
without a frozen association."""
import ctypes as C

import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,height,K,rows,freeze", [
    (320, 240, 3, 0, False),        # blocks of several thousand pixels
    (320, 240, 3, 5000, True),      # more blocks than one scan tile
    (333, 251, 5, 4096, False),     # exactly one tile, ragged pixel tiles
    (40, 30, 1, 0, False),          # nothing to split
])
def test_parts_give_the_gradients_of_whole_blocks(width, height, K, rows, freeze):
    import torch
    from paper_2111_13652_amd import _lib
    from paper_2111_13652_amd.gsdf import GsdfMap, camera, keyframe_loss
    rng = np.random.default_rng(width + K)
    f = 525.0 * width / 640
    cam = synth.Camera(f, f, (width - 1) / 2, (height - 1) / 2, width, height, 0.3, 4.0)
    u, v = np.meshgrid(np.arange(width), np.arange(height))
    D = np.stack([0.5 / (1 - 0.3 * ((u - cam.cx) / cam.fx + 0.4 * (v - cam.cy) / cam.fy))
                  + 0.001 * rng.standard_normal(u.shape) for _ in range(K)]).astype(np.float32)
    eye = np.hstack([np.eye(3), np.zeros((3, 1))])
    G = GsdfMap(0.01, 0.05, 8192)
    G.fuse(dev(D[0]), cam, dev(eye))
    n = max(G.num_blocks(), rows)
    params = G.export_params(n)
    T0 = dev(np.stack([synth.perturb_pose(eye, 3 + i, 0.5, 0.005) for i in range(K)]))
    xi = dev(1e-3 * rng.standard_normal((K, 6)))
    depth = dev(D)
    lib, c = _lib.load(), camera(cam)
    full = lib.gsdf_keyframe_scratch_bytes(C.byref(c), K, n)
    ptr = lambda t: None if t is None else C.c_void_p(t.data_ptr())
    assoc = None
    if freeze:
        assoc = torch.empty((K, height, width, 3), dtype=torch.int32, device="cuda")
        keyframe_loss(G, params, dev(np.zeros((K, 6))), depth, cam, T0, 0.01, assoc)
    out = []
    for size in (full, full - 256, full):
        scratch = torch.randint(0, 255, (full,), dtype=torch.uint8, device="cuda")
        gl = torch.linspace(0.5, 1.5, K, device="cuda")
        dparams, dxi = torch.zeros_like(params), torch.empty_like(xi)
        _lib.check(lib.gsdf_backward(C.byref(G._map), ptr(depth), K, C.byref(c), ptr(T0), ptr(xi), ptr(params), n, 0.01,
                                     ptr(assoc), int(freeze), ptr(gl), ptr(dparams), ptr(dxi), None, ptr(scratch), size,
                                     None), "backward")
        torch.cuda.synchronize()
        out.append((dparams, dxi))
    log(f"case: {width}x{height}, {K} keyframes, {G.num_blocks()} blocks of {n} rows, "
        f"{int((out[0][0] != 0).sum())} gradients")
    assert out[0][0].abs().max() > 0
    for dparams, dxi in out[1:]:
        assert torch.equal(dparams, out[0][0]) and torch.equal(dxi, out[0][1])
    # the gather's sum over the voxels is the loss's derivative in a common psi
    h = 1e-4
    plus, minus = params.clone(), params.clone()
    plus[..., 0] += h
    minus[..., 0] -= h
    w = torch.linspace(0.5, 1.5, K, device="cuda", dtype=torch.float64)
    if freeze:
        diff = (w * (keyframe_loss(G, plus, xi, depth, cam, T0, 0.01, assoc, True)
                     - keyframe_loss(G, minus, xi, depth, cam, T0, 0.01, assoc, True))).sum() / (2 * h)
        got = out[0][0][..., 0].double().sum()
        assert abs(float(diff - got)) <= 1e-2 * float(out[0][0][..., 0].abs().double().sum())
