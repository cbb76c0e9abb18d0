"""That blocks near the camera are fused and gathered in parts at all (the
partial-sum buffers at the end of the scratch are written), and that the
gathered gradients are the pixels' own: against float64 sums over the pixels in
numpy.  A term's float32 residual is within 2e-9 m of the float64 one and a
voxel takes some hundreds of them, far inside 1e-6 of the largest gradient."""
import ctypes as C

import numpy as np
import pytest

from paper_2111_13652_amd import synth
from tests.gpu_helpers import dev, log

pytestmark = pytest.mark.gpu

EYE = np.hstack([np.eye(3), np.zeros((3, 1))])


def _plane(cam, z, rng):
    u, v = np.meshgrid(np.arange(cam.width), np.arange(cam.height))
    d = z / (1 - 0.3 * ((u - cam.cx) / cam.fx + 0.4 * (v - cam.cy) / cam.fy))
    return (d + 0.001 * rng.standard_normal(d.shape)).astype(np.float32)


def _cam(width, height):
    f = 525.0 * width / 640
    return synth.Camera(f, f, (width - 1) / 2, (height - 1) / 2, width, height, 0.3, 4.0)


@pytest.mark.parametrize("storage,width,height,z,split", [
    ("fp32", 640, 480, 0.45, True),
    ("nograd", 333, 251, 0.4, True),
    ("fp32", 333, 251, 0.6, True),
    ("bf16", 40, 30, 2.0, False),
])
def test_fusion_uses_its_buffers(storage, width, height, z, split):
    import torch
    from paper_2111_13652_amd import _lib
    from paper_2111_13652_amd.gsdf import COS_75, GsdfMap, camera
    cam = _cam(width, height)
    lib, c = _lib.load(), camera(cam)
    full = lib.gsdf_integrate_scratch_bytes(C.byref(c))
    pixels = -(-width * height * 16 // 256) * 256
    D, pose = dev(_plane(cam, z, np.random.default_rng(1))), dev(EYE)
    p = _lib.FuseParams(0.01, COS_75)
    maps = []
    for size in (full, pixels):
        scratch = torch.empty((full,), dtype=torch.uint8, device="cuda")
        m = GsdfMap(0.01, 0.05, 8192, storage=storage)
        for _ in range(2):   # the first frame's blocks count few pixels: their slots are not known yet
            scratch.fill_(0xA5)
            _lib.check(lib.gsdf_fuse_frame(C.byref(m._map), D.data_ptr(), C.byref(c), pose.data_ptr(), C.byref(p),
                                           scratch.data_ptr(), size, m.status.data_ptr(), None), "fuse_frame")
        torch.cuda.synchronize()
        used = bool((scratch[pixels:] != 0xA5).any())
        log(f"case: {storage} {width}x{height} at {z} m: {m.num_blocks()} blocks, buffers used: {used}")
        assert m.status_flags() == [] and used == (split and size == full)
        keys = m.keys()
        o = np.lexsort(keys.T[::-1])
        maps.append([keys[o]] + [x[o] for x in m.voxels(len(keys))])
    assert maps[0][3].max() > 0
    for a, b in zip(*maps):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("width,height,K,split", [(320, 240, 3, True), (40, 30, 1, False)])
def test_adjoint_uses_its_buffers(width, height, K, split):
    import torch
    from paper_2111_13652_amd import _lib
    from paper_2111_13652_amd.gsdf import GsdfMap, camera, voxel_order
    rng = np.random.default_rng(width)
    cam, vs, delta = _cam(width, height), 0.01, 0.01
    D = np.stack([_plane(cam, 0.5, rng) for _ in range(K)])
    G = GsdfMap(vs, 0.05, 8192)
    G.fuse(dev(D[0]), cam, dev(EYE))
    n = G.num_blocks()
    params = G.export_params(n)
    T0 = np.stack([synth.perturb_pose(EYE, 3 + i, 0.5, 0.005) for i in range(K)])
    scale = np.linspace(0.5, 1.5, K).astype(np.float32)
    lib, c = _lib.load(), camera(cam)
    full = lib.gsdf_keyframe_scratch_bytes(C.byref(c), K, n)
    scratch = torch.full((full,), 0xA5, dtype=torch.uint8, device="cuda")
    dparams = torch.zeros_like(params)
    xi, dxi = dev(np.zeros((K, 6))), dev(np.zeros((K, 6)))
    depth, T, gl = dev(D), dev(T0), dev(scale)
    _lib.check(lib.gsdf_backward(C.byref(G._map), depth.data_ptr(), K, C.byref(c), T.data_ptr(), xi.data_ptr(),
                                 params.data_ptr(), n, delta, None, 0, gl.data_ptr(), dparams.data_ptr(),
                                 dxi.data_ptr(), None, scratch.data_ptr(), full, None), "backward")
    torch.cuda.synchronize()
    # the buffers of 4 x 512 sums of 8 bytes are the scratch's last region
    pix = K * -(-width // 32) * -(-height // 32) * 1024
    buffers = 2 * pix // max(1024, pix // 2048) + 2
    used = bool((scratch[full - buffers * 16384:][:16384] != 0xA5).any())
    log(f"case: {K} keyframes of {width}x{height}, {n} blocks, buffers used: {used}")
    assert used == split

    # the same gradients from the pixels in float64
    order = np.asarray(voxel_order())
    p = params.cpu().numpy().astype(np.float64)
    Wv = G.weight[: n * 512].view(n, 512).cpu().numpy()
    slot = {tuple(k): i for i, k in enumerate(G.keys())}
    ref = np.zeros((n, 512, 4))
    u, v = np.meshgrid(np.arange(width), np.arange(height))
    for k in range(K):
        d = D[k].astype(np.float64)
        x = np.stack([d * ((u - cam.cx) / cam.fx), d * ((v - cam.cy) / cam.fy), d], -1).reshape(-1, 3)
        q = x @ T0[k][:, :3].T + T0[k][:, 3]
        m = np.floor(q / vs + 0.5).astype(np.int64)
        blocks, inv = np.unique(m >> 3, axis=0, return_inverse=True)
        s = np.array([slot.get(tuple(b), -1) for b in blocks])[inv.reshape(-1)]
        l = m & 7
        c_in = order[l[:, 0] + 8 * l[:, 1] + 64 * l[:, 2]]
        ok = s >= 0
        s, c_in, dq = s[ok], c_in[ok], (q - vs * m)[ok]
        ok = (Wv[s, c_in] > 0) & (np.linalg.norm(p[s, c_in, 1:], axis=-1) > 0)
        s, c_in, dq = s[ok], c_in[ok], dq[ok]
        g = p[s, c_in, 1:]
        ng = np.linalg.norm(g, axis=-1, keepdims=True)
        gh = g / ng
        r = p[s, c_in, 0] + (gh * dq).sum(-1)
        rp = scale[k] * np.clip(r, -delta, delta)
        dg = rp[:, None] * (dq - gh * (gh * dq).sum(-1, keepdims=True)) / ng
        np.add.at(ref, (s, c_in), np.concatenate([rp[:, None], dg], -1))
    got = dparams.cpu().numpy()
    for a, b in ((got[..., :1], ref[..., :1]), (got[..., 1:], ref[..., 1:])):
        assert np.abs(b).max() > 0
        assert (np.abs(a - b) <= 1e-4 * np.abs(b) + 1e-6 * np.abs(b).max()).all()
