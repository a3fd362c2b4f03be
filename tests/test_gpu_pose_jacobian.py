"""The pose gradient at a perturbed view: dL/dxi = J_l(xi)^T times the left-perturbation gradient
at the pose Exp(xi) T, with J_l from the matrix series in binary64, for perturbations from zero
(where the library's vector series ends at once) to a rotation of 3 rad (where its terms grow
before they fall).

Tolerance: both calls render at the same camera up to one rounding of its entries, whose effect on
the gradient stays below the 1e-3 that the parity tests of gradients allow."""
import math

import numpy as np
import pytest
import torch

from tests.gpu_util import DEV, cfg_pair, h, normwise, t
from tests.test_gpu_pose_aux import _cam_at, _hat
from tests.tiny_cases import tiny_case

pytestmark = pytest.mark.gpu


def _left_jacobian(xi):
    ad = np.zeros((6, 6))
    ad[:3, :3] = ad[3:, 3:] = _hat(xi)[:3, :3]
    ad[:3, 3:] = _hat(np.concatenate([np.zeros(3), xi[:3]]))[:3, :3]
    J, P = np.eye(6), np.eye(6)
    for n in range(1, 60):
        P = P @ ad / (n + 1)
        J = J + P
    return J


@pytest.mark.parametrize("size", [0.0, 1e-9, 0.02, 3.0])
def test_pose_gradient_series(size):
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    P.lib()
    case = tiny_case(11, M=60, W=53, H=37, log_scale=-2.4)
    gc, _ = cfg_pair(P, O, eps=0.03)
    d = np.array([0.3, -0.2, 0.25, 0.5, -0.7, 0.4])
    xi = (size / math.sqrt(float((d[3:] ** 2).sum()))) * d  # |phi| = size
    cam0 = _cam_at(case["cam"], -xi)                         # Exp(xi) cam0 = the case's camera
    gd = {k: t(v) for k, v in case["gauss"].items()}
    got = []
    for cam, x in ((cam0, t(xi.reshape(1, 6))), (_cam_at(cam0, np.float32(xi).astype(np.float64)), None)):
        view = P.View(cam, t(case["base_rgb"]), t(case["base_depth"]), t(case["target_rgb"]), t(case["target_depth"]))
        ws = P.Workspace(gc, 60, [cam], device=DEV)
        P.render_fwd(gc, gd, [view], ws, pose_xi=x)
        dpose = torch.zeros(1, 6, device=DEV)
        P.render_bwd(gc, gd, [view], ws, P.zeros_like_gaussians(gd), dpose, pose_xi=x)
        torch.cuda.synchronize()
        got.append(h(dpose)[0].astype(np.float64))
    assert np.linalg.norm(got[1]) > 0
    assert normwise(got[0], _left_jacobian(xi).T @ got[1]) < 1e-3
