"""The Gauss-Newton system at image sizes whose rows do not divide a lane's stride, with several
pixels per lane (more than 262144 pixels), and with a principal point close to 0, where the
shared quotients give way to divisions.  Against the reference, to the tolerance of the parity
tests (a binary32 bound plus what the pairs near a decision can contribute)."""
import pytest

from tests.test_gpu_icp import P, _check_system, _room_pair  # noqa: F401  (P is a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("W,H,corner", [(323, 241, False), (61, 97, False), (701, 399, False), (160, 120, True)])
def test_icp_system_sizes(P, W, H, corner):  # noqa: F811
    camA, DA, camB, DB = _room_pair(W, H)
    if corner:
        camA = {**camA, "cx": 1e-7}
        camB, DB = camA, DA
    _check_system(P, camA, DA, camB, DB, camA["R"], camA["t"], 0.1)
