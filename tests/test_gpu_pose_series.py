"""The series of dL/dxi = J_l(xi)^T g at a view rendered from Exp(xi) T, against J_l from the matrix series
in binary64: the same camera is rendered without xi (the images have to be the same bits, so g is the
same), which leaves one rounding of the result to binary32.  Rotations up to the 2 pi that 39 terms
reach, with translations from nothing to twice them.

Tolerance: half a unit of the last place for the rounding of the result and half a unit for that of g in
the second call, each through J_l^T: 2^-24 (|y| + |J_l^T| |g|), and 1e-12 of that for the series."""
import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, cfg_pair, h, t
from tests.test_gpu_pose_aux import _cam_at
from tests.test_gpu_pose_jacobian import _left_jacobian
from tests.tiny_cases import tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("phi", [1e-9, 0.02, 1.0, 3.0, 6.28])
@pytest.mark.parametrize("rho", [0.0, 0.3, 2.0])
def test_series_to_the_last_place(phi, rho):
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    print(f"pose series: phi={phi} rho={rho}", flush=True)
    case = tiny_case(11, M=60, W=53, H=37, log_scale=-2.4)
    gc, _ = cfg_pair(P, O, eps=0.03)
    gd = {k: t(v) for k, v in case["gauss"].items()}
    rng = np.random.default_rng(int(100 * phi + 10 * rho))
    checked = 0
    for _ in range(8):
        a, b = rng.normal(size=3), rng.normal(size=3)
        xi = np.float32(np.concatenate([rho * a / np.linalg.norm(a), phi * b / np.linalg.norm(b)]))
        cam0 = _cam_at(case["cam"], -xi.astype(np.float64))
        got, images = [], []
        for cam, x in ((cam0, t(xi.reshape(1, 6))), (_cam_at(cam0, xi.astype(np.float64)), None)):
            view = P.View(cam, t(case["base_rgb"]), t(case["base_depth"]), t(case["target_rgb"]), t(case["target_depth"]))
            ws = P.Workspace(gc, 60, [cam], device=DEV)
            P.render_fwd(gc, gd, [view], ws, pose_xi=x)
            dpose = torch.zeros(1, 6, device=DEV)
            P.render_bwd(gc, gd, [view], ws, P.zeros_like_gaussians(gd), dpose, pose_xi=x)
            torch.cuda.synchronize()
            got.append(h(dpose)[0].astype(np.float64))
            images.append((h(view.out_rgb), h(view.out_depth)))
        if not all(np.array_equal(p, q) for p, q in zip(*images)):
            continue  # an entry of the two cameras is rounded differently
        checked += 1
        J = _left_jacobian(xi.astype(np.float64))
        want = J.T @ got[1]
        assert np.abs(got[1]).max() > 0
        tol = (2.0 ** -24 + 1e-12) * (np.abs(want) + np.abs(J.T) @ np.abs(got[1]))
        assert (np.abs(got[0] - want) <= tol).all(), (got[0], want, tol)
    assert checked >= 2
