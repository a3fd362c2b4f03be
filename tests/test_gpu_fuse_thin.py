"""Fusion of a lattice 2 points wide and high and 2^29 + 64 deep, which has more cells than one launch has lanes
for: the points in view at either end of it, with the values of the update formed here (each a few exact
binary32 operations: every number is a small multiple of a power of two), and none beside them."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, h

pytestmark = pytest.mark.gpu


def test_fused_points_of_a_thin_lattice():
    import paper_2509_11574_amd as P
    n, voxel, mu = (1 << 29) + 64, 0.125, 4.0
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 52 GB of device memory")
    print("fuse: 2 x 2 x 2^29 + 64", flush=True)
    vol = P.Volume((2, 2, n), (0.0, 0.0, 0.0), voxel, mu, device=DEV, skip_bricks=False)
    depth, rgb = torch.full((64, 64), 6.0, device=DEV), torch.full((3, 64, 64), 0.5, device=DEV)
    touched = 0
    for at in (4, n - 128):
        z0 = np.float32(at) * np.float32(voxel)
        cam = {"width": 64, "height": 64, "fx": 1.0, "fy": 1.0, "cx": 32.0, "cy": 32.0,
               "R": np.eye(3, dtype=np.float32).reshape(-1), "t": np.float32([0.0, 0.0, -z0])}
        P.fuse(vol, cam, depth, rgb)
        lo = max(at - 200, 0)
        zc = (np.arange(lo, min(at + 400, n)).astype(np.float32) * np.float32(voxel) - z0).astype(np.float32)
        seen = (zc > 0) & (6.0 - zc >= -mu)
        want = np.where(seen, np.minimum(1.0, (6.0 - zc) / mu), 1.0)
        s = slice(4 * lo, 4 * lo + 4 * zc.size)
        np.testing.assert_array_equal(h(vol.weight[s]).reshape(-1, 4), np.repeat(seen[:, None].astype(np.float32), 4, 1))
        np.testing.assert_array_equal(h(vol.tsdf[s]).reshape(-1, 4), np.repeat(want[:, None].astype(np.float32), 4, 1))
        band = seen & (np.abs(6.0 - zc) <= mu)
        np.testing.assert_array_equal(h(vol.rgb[:, s]).reshape(3, -1, 4), np.broadcast_to(0.5 * band[None, :, None], (3, zc.size, 4)))
        assert seen.sum() >= 50
        touched += 4 * int(seen.sum())
    total = sum(int(torch.count_nonzero(vol.weight[k:k + (1 << 28)])) for k in range(0, 4 * n, 1 << 28))
    assert total == touched
