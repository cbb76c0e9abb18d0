"""Surfels into a program's own buffers: a capacity that ends inside a
block, and ids that are only four-byte aligned, give the first rows of the
full cloud and touch nothing behind them; blocks with every subvoxel on the
surface and blocks with none."""
import ctypes as C

import numpy as np
import pytest

from tests.gpu_helpers import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level", [0, 1])
@pytest.mark.parametrize("short,shift", [(0, 0), (1, 1), (700, 3)])
def test_capacity_and_alignment(level, short, shift):
    import torch
    from paper_2111_13652_amd import _lib
    from paper_2111_13652_amd.gsdf import GsdfMap
    rng = np.random.default_rng(level)
    G = GsdfMap(0.01, 0.05, 16)
    keys = np.array([[0, 0, 0], [1, 0, 0], [0, 1, 0], [-1, -2, 3]], np.int32)
    psi = np.zeros((4, 512), np.float32)          # every voxel: all of its subvoxels that a plane leaves
    psi[1] = 0.04                                 # none
    psi[2] = rng.uniform(-0.0095, 0.0095, 512)    # about the selection's limits
    psi[3] = np.where(rng.random(512) < 0.5, 0.0, np.nan)
    g = rng.standard_normal((4, 512, 3)).astype(np.float32)
    W = np.ones((4, 512), np.float32)
    G.import_blocks(keys, psi, g, W)
    p, n, i = G.surfels(level)
    total = len(i)
    cap = total - short
    log(f"case: level {level}, {total} surfels, capacity {cap}, ids {4 * shift} bytes off")
    assert total > 800
    lib = _lib.load()
    pts = torch.full((total, 3), -7.0, device="cuda")
    nrm = torch.full((total, 3), -7.0, device="cuda")
    store = torch.full((4 * total + 4,), -7, dtype=torch.int32, device="cuda")
    ids = store[shift:]
    count = torch.zeros(1, dtype=torch.int64, device="cuda")
    scratch = torch.empty(lib.gsdf_surfel_scratch_bytes(C.byref(G._map)), dtype=torch.uint8, device="cuda")
    _lib.check(lib.gsdf_extract_surfels(C.byref(G._map), level, pts.data_ptr(), nrm.data_ptr(), ids.data_ptr(), cap,
                                        count.data_ptr(), scratch.data_ptr(), scratch.numel(),
                                        torch.cuda.current_stream().cuda_stream), "extract_surfels")
    assert int(count) == total
    assert torch.equal(pts[:cap], p[:cap]) and torch.equal(nrm[:cap], n[:cap])
    assert torch.equal(ids[:4 * cap].reshape(-1, 4), i[:cap])
    assert bool((pts[cap:] == -7).all()) and bool((nrm[cap:] == -7).all())
    assert bool((ids[4 * cap:] == -7).all()) and bool((store[:shift] == -7).all())
