"""hash_raycast allocates the depth ranges only where its march forms them: not for regions and pools that
are marched with the block directory (up to 32768 blocks, a pool of up to 65535)."""
import ctypes

import pytest
import torch

import synth
from tests.gpu_util import DEV, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,capacity,used", [((64, 64, 64), 1024, False), ((256, 256, 256), 65535, False),
                                                ((64, 64, 64), 65536, True), ((264, 256, 256), 1024, True)])
def test_scratch_of_a_hash_raycast(dims, capacity, used):
    import paper_2509_11574_amd as P
    print(f"hash scratch: {dims} {capacity}", flush=True)
    w = synth.workload_small(M=10)
    sc, cam = w["scene"], w["cam"].as_dict()
    vol = P.HashVolume(dims, sc.origin, sc.voxel, sc.trunc, capacity=capacity)
    P.hash_fuse(vol, cam, t(w["depth"]), t(w["rgb"]))
    H, W = cam["height"], cam["width"]
    out = [(torch.empty(H, W, device=DEV), torch.empty(3, H, W, device=DEV))]
    torch.cuda.synchronize()
    before = torch.cuda.memory_allocated()
    torch.cuda.reset_peak_memory_stats()
    P.hash_raycast(vol, [cam], out=out)
    assert (torch.cuda.max_memory_allocated() > before) == used
    n, c = ctypes.c_size_t(7), P.camera(cam)
    s = vol.struct()
    assert P.lib().gps_hash_range_floats(ctypes.byref(s), ctypes.byref(c), 1, ctypes.byref(n)) == 0
    assert n.value == (P.gps.hash_range_floats([cam]) if used else 0)
    assert P.lib().gps_hash_range_floats(ctypes.byref(s), ctypes.byref(c), 0, ctypes.byref(n)) == -1
    assert P.lib().gps_hash_range_floats(ctypes.byref(s), None, 1, ctypes.byref(n)) == -1
    torch.cuda.synchronize()
