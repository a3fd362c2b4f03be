"""Sorting of long tile lists: one tile whose list holds 511 keys (the shortest the buckets
sort), 4096 and 4097 (the most that meet in LDS, and the fewest that are split first), with depths that
are spread, that all coincide (the network, in LDS and in memory; the order is then the Gaussians'),
and that crowd into a hundredth of a millimetre but for a few outliers (full buckets next to empty
ones).  The rendered colour and depth of a list composited to its end depend on its order; compared
with the reference, which sorts by (depth key, index), to the parity tests' 1e-4."""
import numpy as np
import pytest

from tests.gpu_util import cfg_pair, normwise
from tests.test_gpu_edges import _run
from tests.tiny_cases import tiny_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,depths", [(511, "spread"), (4096, "spread"), (4097, "spread"), (1500, "equal"),
                                      (5000, "equal"), (3000, "crowded"), (6000, "crowded")])
def test_long_list_order(n, depths):
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    P.lib()
    O.lib()
    W = H = 16
    case = tiny_case(3, M=n, W=W, H=H, f=30.0, log_scale=-1.2, invalid_frac=0.0, rotate=False)
    rng = np.random.default_rng(n)
    z = rng.uniform(1.0, 2.4, n)
    if depths == "equal":
        z[:] = 1.5
    elif depths == "crowded":
        z = 1.5 + 1e-5 * rng.uniform(size=n)
        z[rng.choice(n, 20, replace=False)] = rng.uniform(1.0, 2.4, 20)
    c = case["cam"]
    u, v = rng.uniform(0, W, n), rng.uniform(0, H, n)
    case["gauss"]["mean"] = np.stack([(u - c["cx"]) / c["fx"] * z, (v - c["cy"]) / c["fy"] * z, z]).astype(np.float32)
    case["gauss"]["opacity_logit"] = rng.normal(-4.5, 0.2, n).astype(np.float32)
    case["base_depth"][:] = 3.0
    gc, oc = cfg_pair(P, O, eps=0.03, T_min=0.0)
    C, D, _, st = _run(P, gc, case, np.ones((3, W * H)), np.ones(W * H))
    assert st["n_instances"] == n and st["n_tiles"] == 1
    r = O.render(oc, case["gauss"], c, case["base_rgb"], case["base_depth"])
    keep = r["flag"] == 0
    assert keep.mean() > 0.5 and r["n"][keep].mean() > 0.2 * n
    assert normwise(C, r["rgb"], keep) < 1e-4
    assert normwise(D, r["depth"], keep) < 1e-4
