"""The order in which the unsorted blend (GPS_RENDER_NO_SORT) adds a list: group k of 64 consecutive
view-Gaussians stands in part k mod 4 of every tile's list, over the views of a call.

One pixel sees all Gaussians with opacity exactly 1/2.  Those of one part have colour B = 2^30, as many
of another -B (their partial sums are exact and cancel) and those of a third 1.  The ones add up without
rounding where they stand behind both, and vanish beside B / 2 otherwise, so each result is one
value, with no tolerance.
"""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, cfg_pair, t

pytestmark = pytest.mark.gpu
B = 2.0 ** 30


def _colours(group, plus, minus, ones):
    part = group % 4
    return np.where(part == plus, B, np.where(part == minus, -B, np.where(part == ones, 1.0, 0.0))).astype(np.float32)


# (plus, minus, ones)
@pytest.mark.parametrize("parts", [(0, 1, 2), (0, 1, 3), (1, 2, 3), (2, 0, 3), (0, 2, 1), (1, 2, 0), (0, 3, 2)])
@pytest.mark.parametrize("M,V", [(448, 1), (700, 1), (150, 3), (600_000, 1)])
def test_the_parts_of_an_unsorted_list(parts, M, V):
    import paper_2509_11574_amd as P
    from oracle import oracle as O

    W = H = 32
    print(f"unsorted order: M={M} V={V} parts={parts}", flush=True)
    cam = {"width": W, "height": H, "fx": 32.0, "fy": 32.0, "cx": 16.0, "cy": 16.0, "R": np.eye(3, dtype=np.float32).reshape(-1),
           "t": np.zeros(3, np.float32)}
    cfg, _ = cfg_pair(P, O, mode=1, no_sort=True)
    z = np.linspace(1.0, 2.0, M, dtype=np.float32)
    seen = (np.arange(M) < 500) | (np.arange(M) >= M - 500)  # (a large map's others are behind the camera)
    z[~seen] *= -1.0
    g = {"mean": np.stack([0 * z, 0 * z, z]), "log_scale": np.full((3, M), np.log(0.02), np.float32),
         "quat": np.tile(np.float32([[1], [0], [0], [0]]), (1, M)), "opacity_logit": np.zeros(M, np.float32)}
    for v in range(V):  # the colours that are telling in view v
        group = (v * M + np.arange(M)) // 64
        c = np.where(seen, _colours(group, *parts), np.float32(0.0))
        n = min((c == B).sum(), (c == -B).sum())  # as many with B as with -B
        for s in (B, -B):
            c[np.nonzero(c == s)[0][n:]] = 0.0
        if n == 0 or (c == 1.0).sum() == 0:
            continue
        g["rgb"] = np.stack([c, c, c])
        views = [P.View(cam, torch.zeros(3, H, W, device=DEV), torch.full((H, W), 5.0, device=DEV)) for _ in range(V)]
        gd = {k: t(x) for k, x in g.items()}
        ws = P.Workspace(cfg, M, [cam] * V, device=DEV)
        P.render_fwd(cfg, gd, views, ws)
        torch.cuda.synchronize()
        assert ws.status() == 0
        ones = float((c == 1.0).sum()) if parts[2] > max(parts[:2]) else 0.0
        # (sum of alpha c) / (1 + sum of alpha), alpha = 1/2, one rounding each as in the blend
        want = np.float32(0.5 * ones) * (np.float32(1.0) / np.float32(1.0 + 0.5 * seen.sum()))
        got = views[v].out_rgb[:, 16, 16].cpu().numpy()
        assert (got == want).all(), (v, got, want)
