"""Insertion of more Gaussians than are searched by sixteen lanes each (32768): those that a capacity of
32768 takes with sixteen lanes are the same bits as the first of the whole set, over masks of every
pixel, of a quarter of the 8x8 blocks, and of few pixels, in frames of ragged sizes."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, h

pytestmark = pytest.mark.gpu
FEW = 32768


@pytest.mark.parametrize("W,H", [(257, 131), (643, 471), (1280, 720)])
@pytest.mark.parametrize("kind", ["all", "blocks", "sparse"])
def test_more_than_few(W, H, kind):
    import paper_2509_11574_amd as P
    print(f"insertion: {W}x{H} {kind}", flush=True)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(W + H)

    def uniform(*s):
        return torch.rand(*s, device=DEV, generator=gen)

    cam = {"width": W, "height": H, "fx": 0.9 * W, "fy": 0.91 * W, "cx": W / 2 - 0.3, "cy": H / 2 + 0.2,
           "R": np.eye(3, dtype=np.float32).reshape(-1), "t": np.float32([0.1, -0.2, 0.3])}
    x, y = torch.arange(W, device=DEV) / W, torch.arange(H, device=DEV)[:, None] / H
    depth = (1.5 + 0.6 * torch.sin(7 * x) * torch.cos(5 * y) + 0.002 * uniform(H, W)).masked_fill(uniform(H, W) < 0.02, 0.0)
    mask = {"all": torch.ones(H, W, device=DEV), "sparse": (uniform(H, W) < 0.06).float(),
            "blocks": (uniform((H + 7) // 8, (W + 7) // 8) < 0.25).float().repeat_interleave(8, 0).repeat_interleave(8, 1)[:H, :W]}[kind]
    frame = uniform(3, H, W)
    args = (cam, (frame + mask).contiguous(), frame, torch.zeros(H, W, device=DEV), depth.contiguous(), uniform(H, W))
    few, pix, n = P.insert_gaussians(*args, fraction=1.0, capacity=FEW)
    every, pixels, total = P.insert_gaussians(*args, fraction=1.0)
    torch.cuda.synchronize()
    assert total > FEW or (kind != "all" and (W, H) != (1280, 720))
    k = min(total, FEW)
    assert torch.equal(pix[:k], pixels[:k])
    for name, v in few.items():
        a, b = h(v).reshape(-1, v.shape[-1])[:, :k], h(every[name]).reshape(-1, every[name].shape[-1])[:, :k]
        np.testing.assert_array_equal(a, b, err_msg=name)
    assert float(every["log_scale"].std()) > 0
