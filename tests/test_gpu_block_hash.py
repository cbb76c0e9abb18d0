"""Block lookup where the hash has least to spare: tables filled to the last
slot, and keys at the ends of their 21-bit range.  Every block that went in
is found again: a second import writes new values into the same slots."""
import numpy as np
import pytest

from paper_2111_13652_amd.gsdf import GsdfMap, voxel_order

pytestmark = pytest.mark.gpu


def _keys(kind, n):
    i = np.arange(n)
    if kind == "corners":
        ends = np.array([-(1 << 20), -(1 << 20) + 1, -1, 0, 1, (1 << 20) - 3, (1 << 20) - 2])   # the range of keys
        k = np.stack(np.meshgrid(ends, ends, ends), -1).reshape(-1, 3)
        return k[:n]
    if kind == "line":
        return np.stack([i - n // 2, 0 * i, 0 * i], 1)
    s = 4096   # a lattice whose keys share their low 12 bits
    return np.stack([i % 8, i // 8 % 8, i // 64], 1) * s - 2 * s


@pytest.mark.parametrize("kind,n,slots", [("corners", 256, 256), ("line", 256, 256), ("lattice", 255, 256),
                                          ("lattice", 300, 512), ("corners", 1, 16)])
def test_every_block_is_found_again(kind, n, slots):
    keys = _keys(kind, n).astype(np.int32)
    assert len(np.unique(keys, axis=0)) == len(keys) == n
    G = GsdfMap(0.02, 0.1, n, hash_slots=slots)
    order = voxel_order()
    rng = np.random.default_rng(n)
    g = np.zeros((n, 512, 3), np.float32)
    g[..., 2] = 1.0
    W = np.ones((n, 512), np.float32)
    for _ in range(2):
        psi = rng.uniform(-0.05, 0.05, (n, 512)).astype(np.float32)
        G.import_blocks(keys, psi, g, W)
        assert not G.status_flags()
        assert G.num_blocks() == n
        got = G.keys()
        a, b = np.lexsort(got.T), np.lexsort(keys.T)
        assert np.array_equal(got[a], keys[b])
        out = G.export_params(n).cpu().numpy()[:, order, 0]
        assert np.array_equal(out[a], psi[b])
