"""Fusion skips cells of lattice points that lie outside the view.  The set of points it reaches is
the reference's (weights equal, no tolerance) for lattices whose rows are not whole cells, and
cameras inside the lattice, beside it, looking past it or away, with the principal point outside
the image, a mirrored axis, and a lattice far from the origin (where the points' rounding is
largest); the values to the parity tests' 2e-5, far from the origin plus the binary32 rounding of a depth:
six operations of the size of the point's and the camera's coordinates, over the truncation."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, h, t
from tests.tiny_cases import rot_xyz

pytestmark = pytest.mark.gpu

KINDS = ("inside", "beside", "away", "corner", "mirrored", "far")


@pytest.mark.parametrize("dims", [(2, 2, 2), (3, 50, 40), (17, 20, 35), (65, 30, 21), (100, 33, 26), (192, 40, 12)])
@pytest.mark.parametrize("kind", KINDS)
def test_fused_points(dims, kind):
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    P.lib()
    rng = np.random.default_rng(sum(dims) + 1000 * KINDS.index(kind))
    voxel, W, H = 0.05, 71, 53
    origin = np.array([-600.0, 350.0, 200.0]) if kind == "far" else np.array([-0.4, 0.1, 0.2])
    size = voxel * np.array(dims)
    touched = 0
    for _ in range(4):
        centre = origin + size * rng.uniform(0.3, 0.7, 3)
        if kind in ("beside", "away"):
            centre = origin + size * rng.uniform(1.2, 2.0, 3)
        R = rot_xyz(*rng.uniform(-3.0, 3.0, 3))
        if kind == "beside":  # towards the lattice, off its middle
            z = (origin + size * rng.uniform(0.0, 1.0, 3) - centre)
            z /= np.linalg.norm(z)
            x = np.cross(z, [0.3, 1.0, 0.2])
            x /= np.linalg.norm(x)
            R = np.stack([x, np.cross(z, x), z])
        f = rng.uniform(20.0, 90.0)
        cam = {"width": W, "height": H, "fx": float(np.float32(-f if kind == "mirrored" else f)), "fy": float(np.float32(f * 1.1)),
               "cx": float(np.float32(-40.0 if kind == "corner" else 34.7)), "cy": float(np.float32(70.0 if kind == "corner" else 26.2)),
               "R": R.astype(np.float32), "t": (-R @ centre).astype(np.float32)}
        depth = rng.uniform(0.5, 4.0, (H, W)).astype(np.float32)
        rgb = rng.uniform(0, 1, (3, H, W)).astype(np.float32)
        grid = O.make_grid(dims, tuple(origin), voxel, 0.3, 100.0)
        ref = O.new_volume(grid)
        vol = P.Volume(dims, tuple(origin), voxel, 0.3, device=DEV)
        O.fuse(grid, ref, cam, depth, rgb)
        P.fuse(vol, cam, t(depth), t(rgb))
        torch.cuda.synchronize()
        np.testing.assert_array_equal(h(vol.weight), ref["weight"].astype(np.float32))
        np.testing.assert_array_equal(h(vol.rgb_weight), ref["rgb_weight"].astype(np.float32))
        tol = 2e-5
        if kind == "far":
            tol += 6 * 2.0**-24 * (np.abs(origin).sum() + size.sum() + np.abs(cam["t"]).max()) / 0.3
        assert np.abs(h(vol.tsdf) - ref["tsdf"]).max() < tol
        assert np.abs(h(vol.rgb) - ref["rgb"]).max() < 2e-5
        touched += int((ref["weight"] > 0).sum())
    assert touched > 0 or dims == (2, 2, 2) or kind == "away"
