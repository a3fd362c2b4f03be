"""The hashed raycast with table lookups (a pool too large for a directory entry, a region of more than
32768 blocks), with and without depth ranges and block minima, against the reference and, bitwise,
against the dense raycast of the same lattice; the number of launches tells which route ran."""
import pytest
import torch

import synth
from tests.gpu_util import t
from tests.test_gpu_hash import _check_volume, _raycast_checks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,voxel,capacity", [((64, 64, 64), 0.02, 65536), ((272, 264, 248), 0.0047, 4096)])
def test_table_route_against_dense_and_reference(dims, voxel, capacity):
    import paper_2509_11574_amd as P
    from oracle import oracle as O
    print(f"hash table route: {dims} {capacity}", flush=True)
    w = synth.workload_small(M=10)
    sc, cam = w["scene"], w["cam"].as_dict()
    vol = P.HashVolume(dims, sc.origin, voxel, 4 * voxel, capacity=capacity)
    P.hash_fuse(vol, cam, t(w["depth"]), t(w["rgb"]))
    torch.cuda.synchronize()
    assert vol.state()["status"] == 0
    grid = O.make_grid(dims, sc.origin, voxel, 4 * voxel, 100.0)
    mask = O.alloc_blocks(grid, cam, w["depth"])
    ref = O.fuse(grid, O.new_volume(grid), cam, w["depth"], w["rgb"], block_mask=mask)
    _check_volume(O, vol, grid, ref, mask, 2e-5)
    for ranged, launches in ((True, 3), (False, 1)):
        P.gps.profile_start()
        P.hash_raycast(vol, [cam], range_scratch=ranged)
        torch.cuda.synchronize()
        assert P.gps.profile_read()["raycast"][0] == launches
        P.gps.profile_stop()
    near = dict(cam, width=101, height=67, cx=50.0, cy=33.0)
    _raycast_checks(P, O, vol, grid, dims, [cam, near], ref["tsdf"].astype("float32"), ref["rgb"].astype("float32"))
