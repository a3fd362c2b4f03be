"""Insertion with few, far apart mask pixels and a cap out of reach: the search walks rings of up to
a hundred and more 8x8 blocks (several batches of a search group's sixteen lanes), for numbers of
new Gaussians around the sixteen that share a block, on a frame whose last blocks are cut.

Tolerances are those of the insertion parity tests (binary32 distances of vertices up to 2 m
apart: log-scales within 1e-4)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_mask", [15, 16, 17, 33])
def test_insertion_wide_rings(n_mask):
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    W, H = 203, 141
    rng = np.random.default_rng(n_mask)
    cam = {"width": W, "height": H, "fx": 150.0, "fy": 150.0, "cx": W / 2, "cy": H / 2,
           "R": np.eye(3, dtype=np.float32), "t": np.zeros(3, np.float32)}
    D = rng.uniform(1.0, 1.6, (H, W)).astype(np.float32)
    K = np.zeros((3, H, W), np.float32)
    C = K.copy()
    C.reshape(3, -1)[:, rng.choice(W * H, n_mask, replace=False)] = 0.5
    z = np.zeros((H, W), np.float32)
    want, wpix = O.insert_gaussians(cam, C, K, z, D, z, scale_cap=10.0)
    out, pix, n_taken = P.insert_gaussians(cam, t(C), t(K), t(z), t(D), t(z), scale_cap=10.0)
    torch.cuda.synchronize()
    assert n_taken == wpix.size == n_mask
    np.testing.assert_array_equal(pix.cpu().numpy(), wpix)
    np.testing.assert_allclose(out["log_scale"].cpu().numpy(), want["log_scale"], rtol=0, atol=1e-4)
    np.testing.assert_allclose(out["mean"].cpu().numpy(), want["mean"], rtol=0, atol=4e-6)
