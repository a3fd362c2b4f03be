"""Binning of maps whose wavefronts take several shares (more than 524288 view-Gaussians, or fewer rows of counts
than blocks), by LDS counters and by shared rows: most Gaussians lie behind the cameras, and images and
gradients are the same bits as those of the map of the seen ones alone, zero for the others.  And of a view
of more than 12288 tiles, whose counters are always the shared rows: the image is the same bits as
with larger tiles, the gradients the same sums in another order (a sum over a few hundred pixels
of terms of either sign, relative to the largest of its attribute: 1e-4)."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, h, t
from tests.tiny_cases import tiny_case

pytestmark = pytest.mark.gpu


def _spread(case, M, rng):
    """The case's Gaussians at ascending random places of a map of M, the others behind the camera."""
    g, c = case["gauss"], case["cam"]
    at = np.sort(rng.choice(M, g["opacity_logit"].size, replace=False))
    back = rng.normal(size=(3, M)) * 0.1 + np.array([[0.0], [0.0], [-2.0]])
    back = c["R"].astype(np.float64).reshape(3, 3).T @ (back - c["t"].astype(np.float64).reshape(3, 1))
    big = {}
    for k, v in g.items():
        big[k] = np.repeat(v[..., :1], M, axis=-1) if k != "mean" else back.astype(np.float32)
        big[k][..., at] = v
        big[k] = np.ascontiguousarray(big[k])
    return big, at


def _render(P, case, g, V, tile, cap, ups):
    gd = {k: t(v) for k, v in g.items()}
    cfg = P.RenderCfg(tile_w=tile[0], tile_h=tile[1], batch=tile[2], pix_per_thread=tile[3], eps_cull=0.03, max_instances=cap)
    views = [P.View(case["cam"], t(case["base_rgb"]), t(case["base_depth"])) for _ in range(V)]
    ws = P.Workspace(cfg, g["opacity_logit"].size, [case["cam"]] * V, device=DEV)
    ws.buf.fill_(0xFF)
    ws.reset()
    P.gps.profile_start()
    P.render_fwd(cfg, gd, views, ws)
    P.gps.profile_stop()
    scans = P.gps.profile_read()["scan"][0]
    grads = P.zeros_like_gaussians(gd)
    P.render_bwd(cfg, gd, views, ws, grads, dL_drgb=[u[0] for u in ups], dL_ddepth=[u[1] for u in ups])
    torch.cuda.synchronize()
    st = ws.stats()
    assert st["status"] == 0
    return [(h(v.out_rgb), h(v.out_depth)) for v in views], {k: h(v) for k, v in grads.items()}, scans, st


def _upstream(rng, W, H, V):
    return [(t(rng.normal(size=(3, H, W))), t(rng.normal(size=(H, W)))) for _ in range(V)]


# room: rows of counts a view that the capacity has place for (0: shared rows)
@pytest.mark.parametrize("M,V,seen,room", [(600_000, 1, 700, 2000), (600_000, 4, 700, 600), (600_000, 4, 700, 0),
                                           (600_000, 4, 700, 70), (17_000, 1, 300, 65), (17_000, 1, 300, 64)])
def test_several_shares_a_wavefront(M, V, seen, room):
    import paper_2509_11574_amd as P
    print(f"shares: M={M} V={V} room={room}", flush=True)
    W, H = 160, 112
    rng = np.random.default_rng(M + V + room)
    case = tiny_case(5, M=seen, W=W, H=H, f=150.0, log_scale=-3.2)
    big, at = _spread(case, M, rng)
    ups = _upstream(rng, W, H, V)
    n_tiles = 70 * V
    cap = room * n_tiles if room else 64 * n_tiles - 1
    want, want_g, _, _ = _render(P, case, case["gauss"], V, (16, 16, 256, 1), 1 << 20, ups)
    got, got_g, scans, st = _render(P, case, big, V, (16, 16, 256, 1), cap, ups)
    assert st["n_tiles"] == n_tiles and scans == (1 if room else 2), "the counters that the case is for"
    for a, b in zip(got, want):
        np.testing.assert_array_equal(a[0], b[0])
        np.testing.assert_array_equal(a[1], b[1])
    for k, v in got_g.items():
        np.testing.assert_array_equal(v[..., at], want_g[k])
        v[..., at] = 0.0
        assert not v.any(), k
    assert all(np.abs(v).max() > 0 for v in want_g.values())


@pytest.mark.parametrize("M", [300, 20_000])
def test_a_view_of_many_tiles(M):
    import paper_2509_11574_amd as P
    print(f"many tiles: M={M}", flush=True)
    W, H = 1031, 1023
    rng = np.random.default_rng(M)
    case = tiny_case(6, M=M, W=W, H=H, f=900.0, log_scale=-4.0)
    ups = _upstream(rng, W, H, 1)
    got, got_g, scans, st = _render(P, case, case["gauss"], 1, (8, 8, 128, 1), 1 << 22, ups)
    want, want_g, scans16, _ = _render(P, case, case["gauss"], 1, (16, 16, 256, 1), 1 << 22, ups)
    assert st["n_tiles"] == 129 * 128 and (scans, scans16) == (2, 1)
    np.testing.assert_array_equal(got[0][0], want[0][0])
    np.testing.assert_array_equal(got[0][1], want[0][1])
    for k, v in got_g.items():
        assert np.abs(v - want_g[k]).max() <= 1e-4 * np.abs(want_g[k]).max(), k
