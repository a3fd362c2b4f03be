"""Small grids are composited with one pixel per lane whatever pix_per_thread asks (fewer
instructions on the longest list), large ones as asked.  An image of each tile shape on either side
of the limits (16384 wavefronts; backward of tiles of 512 pixels 10240): the pixels are the same bits with 1, 2
and 4 pixels per lane, the gradients the same sums in another order.  A gradient is a sum over a few
hundred pixels of terms of either sign, taken relative to the largest of its attribute: 1e-4."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, h, t
from tests.tiny_cases import tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H", [(90, 70), (1023, 639), (1023, 767), (1024, 1023), (1280, 1000)])
@pytest.mark.parametrize("mode", [0, 1])
def test_pixels_per_lane_agree(W, H, mode):
    import paper_2509_11574_amd as P
    P.lib()
    case = tiny_case(9, M=4000, W=W, H=H, f=0.9 * W, log_scale=-3.6)
    rng = np.random.default_rng(W)
    gC, gD = t(rng.normal(size=(3, H, W))), t(rng.normal(size=(H, W)))
    gd = {k: t(v) for k, v in case["gauss"].items()}
    for shape in ((16, 16), (16, 32), (32, 16)):
        got = {}
        for tile in [c for c in P.gps.TILE_CONFIGS if c[:2] == shape]:
            cfg = P.RenderCfg(tile_w=tile[0], tile_h=tile[1], batch=tile[2], pix_per_thread=tile[3], mode=mode, eps_cull=0.03)
            view = P.View(case["cam"], t(case["base_rgb"]), t(case["base_depth"]))
            ws = P.Workspace(cfg, 4000, [view.cam], device=DEV)
            P.render_fwd(cfg, gd, [view], ws)
            grads = P.zeros_like_gaussians(gd)
            P.render_bwd(cfg, gd, [view], ws, grads, dL_drgb=[gC], dL_ddepth=[gD])
            torch.cuda.synchronize()
            assert ws.stats()["status"] == 0
            got[tile] = (h(view.out_rgb), h(view.out_depth), {k: h(v) for k, v in grads.items()})
        first = next(iter(got.values()))
        for tile, (C, D, G) in got.items():
            assert np.array_equal(C, first[0]) and np.array_equal(D, first[1]), tile
            for k, v in G.items():
                assert np.abs(v - first[2][k]).max() <= 1e-4 * np.abs(first[2][k]).max(), (tile, k)
