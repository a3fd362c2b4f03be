"""Tile binning.  Its blocks count instances per tile in LDS, or, when the capacity leaves no room
for a row of counts per block, in memory; both routes give the same bits, from a workspace whose
every word but the header was NaN.  Sizes around a wavefront's and a block's share, several
iterations per wavefront (M = 300000, most of it behind the camera), Gaussians of more tiles than have bits, and
tiles whose lists end early (opaque Gaussians), whose unread slots count as zero."""
import numpy as np
import pytest
import torch

from paper_2509_11574_amd import gps
from tests.gpu_util import DEV, cfg_pair, h, normwise, t
from tests.tiny_cases import tiny_case

pytestmark = pytest.mark.gpu

W, H = 203, 117


def _case(M, seen, kind):
    case = tiny_case(5, M=seen, W=W, H=H, f=150.0, log_scale=-2.2 if kind == "wide" else -3.4)
    g = case["gauss"]
    if kind == "opaque":
        g["opacity_logit"] = np.full(seen, 6.0, np.float32)
        g["log_scale"] += 1.4
        case["base_depth"][:] = 4.0
    if M > seen:  # the others behind the camera, the seen ones spread over the map
        rng = np.random.default_rng(M)
        c = case["cam"]
        back = rng.normal(size=(3, M)) * 0.1 + np.array([[0.0], [0.0], [-2.0]])
        back = c["R"].astype(np.float64).T @ (back - c["t"].astype(np.float64)[:, None])
        at = np.sort(rng.choice(M, seen, replace=False))
        big = {"mean": back.astype(np.float32)}
        for k, v in g.items():
            if k != "mean":
                big[k] = np.repeat(v[..., :1], M, axis=-1)
            big[k][..., at] = v
        case["gauss"] = {k: np.ascontiguousarray(v) for k, v in big.items()}
    return case


def _route(P, gc, case, gC, gD):
    view = P.View(case["cam"], t(case["base_rgb"]), t(case["base_depth"]))
    gd = {k: t(v) for k, v in case["gauss"].items()}
    ws = P.Workspace(gc, case["gauss"]["opacity_logit"].size, [view.cam], device=DEV)
    ws.buf.fill_(0xFF)
    ws.reset()
    gps.profile_start()
    P.render_fwd(gc, gd, [view], ws)
    gps.profile_stop()
    scans = gps.profile_read()["scan"][0]
    grads = P.zeros_like_gaussians(gd)
    dpose = torch.zeros(1, 6, device=DEV)
    P.render_bwd(gc, gd, [view], ws, grads, dpose, dL_drgb=[gC], dL_ddepth=[gD])
    torch.cuda.synchronize()
    st = ws.stats()
    assert st["status"] == 0
    out = {k: h(v) for k, v in grads.items()}
    out.update(pose=h(dpose), rgb_out=h(view.out_rgb), depth_out=h(view.out_depth))
    return out, st, scans


@pytest.mark.parametrize("M,seen,kind,tile", [(1, 1, "", (16, 16, 256, 1)), (63, 12, "", (16, 32, 128, 2)),
                                              (64, 2, "wide", (8, 8, 128, 1)), (257, 25, "", (16, 16, 256, 1)),
                                              (3000, 40, "wide", (8, 8, 128, 1)), (3000, 30, "opaque", (16, 16, 256, 1)),
                                              (17000, 500, "", (16, 32, 128, 2)), (300000, 800, "", (16, 16, 256, 1))])
def test_routes_agree(M, seen, kind, tile):
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    P.lib()
    O.lib()
    case = _case(M, seen, kind)
    rng = np.random.default_rng(M)
    gC, gD = t(rng.normal(size=(3, H, W))), t(rng.normal(size=(H, W)))
    gc, oc = cfg_pair(P, O, eps=0.03, tile=tile)
    a, sa, na = _route(P, gc, case, gC, gD)
    blocks = min((M + 255) // 256, 64)
    no_room, _ = cfg_pair(P, O, eps=0.03, tile=tile, max_instances=blocks * sa["n_tiles"] - 1)
    assert sa["n_instances"] <= blocks * sa["n_tiles"] - 1, "the case fits the capacity of the second route"
    b, sb, nb = _route(P, no_room, case, gC, gD)
    assert (na, nb) == (1, 2), "the second route clears its rows first"
    assert sa["n_instances"] == sb["n_instances"] and sa["pairs_contrib"] == sb["pairs_contrib"]
    for k in a:
        assert np.isfinite(a[k]).all(), k
        assert np.array_equal(a[k], b[k]), k
    if M <= 3000:
        r = O.render(oc, case["gauss"], case["cam"], case["base_rgb"], case["base_depth"])
        keep = r["flag"] == 0
        assert normwise(a["rgb_out"].reshape(3, -1), r["rgb"], keep) < 1e-4
        assert normwise(a["depth_out"].reshape(-1), r["depth"], keep) < 1e-4


def test_capacity_overflow_routes():
    """One slot short of what is needed: reported, the gradients zero."""
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    P.lib()
    case = _case(3000, 500, "")
    gc, _ = cfg_pair(P, O, eps=0.03)
    zero = torch.zeros(3, H, W, device=DEV)
    _, st, _ = _route(P, gc, case, zero, zero[0].contiguous())
    short, _ = cfg_pair(P, O, eps=0.03, max_instances=st["n_instances"] - 1)
    view = P.View(case["cam"], t(case["base_rgb"]), t(case["base_depth"]))
    gd = {k: t(v) for k, v in case["gauss"].items()}
    ws = P.Workspace(short, 3000, [view.cam], device=DEV)
    ws.buf.fill_(0xFF)
    ws.reset()
    P.render_fwd(short, gd, [view], ws)
    grads = P.zeros_like_gaussians(gd)
    P.render_bwd(short, gd, [view], ws, grads, dL_drgb=[zero + 1.0], dL_ddepth=[zero[0] + 1.0])
    torch.cuda.synchronize()
    assert ws.status() != 0
    assert all(float(v.abs().max()) == 0.0 for v in grads.values())
