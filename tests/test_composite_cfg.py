"""Which configuration the compositing runs with (gps_render_composite_cfg, a host call) on either side of
each line of the rule, and that the autotuner times each set of kernels once."""
from types import SimpleNamespace

import numpy as np
import pytest


@pytest.fixture(scope="module")
def P():
    import paper_2509_11574_amd as P
    P.lib()
    return P


def _cam(W, H):
    return {"width": W, "height": H, "fx": 50.0, "fy": 50.0, "cx": W / 2, "cy": H / 2, "R": np.eye(3), "t": np.zeros(3)}


def _shapes(P, tile, M, *cams):
    cfg = P.RenderCfg(tile_w=tile[0], tile_h=tile[1], batch=tile[2], pix_per_thread=tile[3])
    return tuple((x.batch, x.pix_per_thread) for x in P.gps.composite_cfgs(cfg, M, cams))


# wavefronts at one pixel a lane: W H / 64 for whole tiles
@pytest.mark.parametrize("W,H,M,fwd,bwd", [
    (640, 512, 0, 1, 1),          # 5120: whatever the Gaussians
    (640, 544, 5439, 2, 2),       # 5440, fewer than one a wavefront
    (640, 544, 5440, 2, 1),       # one
    (640, 544, 3 * 5440 - 1, 2, 1),
    (640, 544, 3 * 5440, 1, 1),   # three
    (1024, 640, 100000, 1, 1),    # 10240
    (1024, 672, 100000, 1, 2),    # 10752
    (1024, 1024, 100000, 1, 2),   # 16384
    (1024, 1056, 1000000, 2, 2),  # 16896
])
@pytest.mark.parametrize("tile", [(16, 32, 128, 2), (16, 32, 512, 4), (32, 16, 256, 2)])
def test_lines_of_the_small_grid_rule(P, tile, W, H, M, fwd, bwd):
    asked = (tile[2], tile[3])
    f, b = _shapes(P, tile, M, _cam(W, H))
    assert f == ((256, 1) if fwd == 1 else asked) and b == ((128, 1) if bwd == 1 else asked)
    # the same over two views
    if H % 64 == 0:
        assert _shapes(P, tile, M // 2 + M % 2, _cam(W, H // 2), _cam(W, H // 2)) == (f, b)


def test_tiles_of_256_pixels_and_one_pixel_asked(P):
    assert _shapes(P, (16, 16, 512, 4), 100000, _cam(1024, 1024)) == ((256, 1), (256, 1))
    assert _shapes(P, (16, 16, 512, 4), 100000, _cam(1040, 1024)) == ((512, 4), (512, 4))
    for tile in ((8, 8, 512, 1), (16, 16, 128, 1), (16, 32, 128, 1)):
        assert _shapes(P, tile, 100000, _cam(320, 240)) == ((tile[2], 1), (tile[2], 1))


def test_refused_arguments(P):
    with pytest.raises(P.GpsError):
        _shapes(P, (16, 16, 100, 1), 10, _cam(64, 48))
    with pytest.raises(P.GpsError):
        _shapes(P, (16, 16, 256, 1), -1, _cam(64, 48))
    with pytest.raises(P.GpsError):
        _shapes(P, (16, 16, 256, 1), 10, _cam(0, 48))


def test_autotune_times_each_set_of_kernels_once(P, monkeypatch):
    from paper_2509_11574_amd import autotune
    timed = []

    def time_config(c, params, views, reps):
        timed.append((c.tile_w, c.tile_h, c.batch, c.pix_per_thread))
        return 10.0 - len(timed)  # a later one faster

    monkeypatch.setattr(autotune, "time_config", time_config)
    monkeypatch.setattr(autotune, "shape_key", lambda *a: "k")
    params = {"opacity_logit": SimpleNamespace(numel=lambda: 100000)}
    for W, H, distinct in ((320, 240, 8), (1600, 1600, 19)):
        timed.clear()
        best, ms = autotune.autotune(P.RenderCfg(), params, [SimpleNamespace(cam=_cam(W, H))], use_cache=False)
        assert len(timed) == len(set(timed)) == distinct and len(ms) == len(P.TILE_CONFIGS)
        assert ms[f"{best.tile_w}x{best.tile_h}x{best.batch}x{best.pix_per_thread}"] == min(ms.values())
