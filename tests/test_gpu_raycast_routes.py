"""Two properties of the dense raycast that hold bit for bit:

* Jumping over positive bricks does not change the image, for steps from a fifth of a voxel to five
  voxels and a lattice away from the origin (the exit of a box and the samples' own positions are
  then rounded more coarsely).
* The 32-bit indexing of a stencil and the general one (lattices whose rows are too many for it) read
  the same values: a lattice embedded in a larger one, seen by a camera inside both, gives the same
  image."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import DEV, h, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shift", [0.0, 10.0])
@pytest.mark.parametrize("step", [0.0, 0.004, 0.1])
def test_raycast_skipping_changes_nothing(step, shift):
    import paper_2509_11574_amd as P
    w = synth.workload_small(M=10)
    sc, cam = w["scene"], w["cam"].as_dict()
    d = np.array([shift, -0.7 * shift, 0.5 * shift])
    cam["t"] = (cam["t"].astype(np.float64) - cam["R"].astype(np.float64) @ d).astype(np.float32)
    origin = tuple(np.asarray(sc.origin) + d)
    vol = P.Volume(sc.dims, origin, sc.voxel, sc.trunc, device=DEV)
    P.fuse(vol, cam, t(w["depth"]), t(w["rgb"]))
    keep = vol.brick_min
    (d0, c0), = P.raycast(vol, [cam], step=step)
    vol.brick_min = None
    (d1, c1), = P.raycast(vol, [cam], step=step)
    vol.brick_min = keep
    torch.cuda.synchronize()
    assert int((d0 > 0).sum()) > 100
    np.testing.assert_array_equal(h(d0), h(d1))
    np.testing.assert_array_equal(h(c0), h(c1))


def test_raycast_wide_lattice():
    import paper_2509_11574_amd as P
    n, big, voxel = (8, 40, 48), (8, 4096, 4097), 0.02
    rng = np.random.default_rng(3)
    z, y, x = np.meshgrid(*(np.arange(k) for k in n[::-1]), indexing="ij")
    tsdf = np.clip((30.0 + 4.0 * np.sin(0.3 * y) + 0.5 * x - z) / 4.0, -1.0, 1.0).astype(np.float32)
    rgb = rng.uniform(size=(3,) + tsdf.shape).astype(np.float32)
    cam = {"width": 75, "height": 61, "fx": 90.0, "fy": 90.0, "cx": 37.0, "cy": 30.0, "R": np.eye(3, dtype=np.float32),
           "t": -np.array([0.07, 0.4, 0.05], np.float32)}
    images = []
    for dims in (n, big):
        vol = P.Volume(dims, (0.0, 0.0, 0.0), voxel, 4 * voxel, device=DEV)
        vol.tsdf.view(dims[::-1])[:n[2], :n[1], :n[0]] = t(tsdf)
        vol.rgb.view((3,) + dims[::-1])[:, :n[2], :n[1], :n[0]] = t(rgb)
        (d, c), = P.raycast(vol, [cam], z_near=0.05)
        torch.cuda.synchronize()
        images.append((h(d), h(c)))
        del vol
    hit = images[0][0] > 0
    assert hit.sum() > 100
    np.testing.assert_array_equal(images[0][0][hit], images[1][0][hit])
    np.testing.assert_array_equal(images[0][1][:, hit], images[1][1][:, hit])
