"""The tile ranges and the queue of tiles on either side of the tile counts at which the scan takes
another number of tiles a lane, and passes: the image of a view in tiles of 8x8 is the same bits as
in tiles of 16x16."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, h, t
from tests.tiny_cases import tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tx,ty", [(64, 32), (683, 3), (64, 64), (241, 17), (128, 64), (2731, 3)])  # 2048, 2049, 4096, ...
def test_ranges_of_many_tiles(tx, ty):
    import paper_2509_11574_amd as P
    W, H, M = 8 * tx - 3, 8 * ty - 1, 3000
    print(f"scan of tiles: {tx} x {ty}", flush=True)
    case = tiny_case(12, M=M, W=W, H=H, f=0.9 * max(W, H), log_scale=-4.6)
    gd = {k: t(v) for k, v in case["gauss"].items()}
    got = []
    for tile in (8, 16):
        cfg = P.RenderCfg(tile_w=tile, tile_h=tile, batch=256, eps_cull=0.03, max_instances=1 << 22)
        view = P.View(case["cam"], t(case["base_rgb"]), t(case["base_depth"]))
        ws = P.Workspace(cfg, M, [view.cam], device=DEV)
        ws.buf.fill_(0xFF)
        ws.reset()
        P.render_fwd(cfg, gd, [view], ws)
        torch.cuda.synchronize()
        st = ws.stats()
        assert st["status"] == 0 and (tile == 16 or st["n_tiles"] == tx * ty)
        got.append((h(view.out_rgb), h(view.out_depth), st["pairs_contrib"]))
    np.testing.assert_array_equal(got[0][0], got[1][0])
    np.testing.assert_array_equal(got[0][1], got[1][1])
    assert got[0][2] == got[1][2] > 1000
