"""The hashed raycast with the block directory in LDS against the one with table lookups (taken when
the pool is larger than a directory entry can name): bitwise the same depth and colour over regions
whose rows of blocks end inside a word, fill one, and run over into a second, with and without the
block minima, for two views of different, ragged sizes, and for a pool that overflowed."""
import numpy as np
import pytest
import torch

import synth
from tests.gpu_util import DEV, h, t

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,voxel,capacity", [((64, 64, 64), 0.02, 1024), ((71, 50, 93), 0.015, 2048),
                                                 ((256, 24, 40), 0.005, 2048), ((267, 40, 33), 0.005, 1024),
                                                 ((64, 64, 64), 0.02, 37)])
def test_hash_directory_against_table(dims, voxel, capacity):
    import paper_2509_11574_amd as P
    P.lib()
    w = synth.workload_small(M=10)
    cam = w["cam"].as_dict()
    near = dict(cam, width=101, height=67, cx=50.0, cy=33.0)
    origin = tuple(0.63 - 0.5 * voxel * n for n in dims)  # about the scene's centre
    vols = []
    for cap in (capacity, 65535 + 1):
        vol = P.HashVolume(dims, origin, voxel, 4 * voxel, capacity=cap)
        P.hash_fuse(vol, cam, t(w["depth"]), t(w["rgb"]))
        vols.append(vol)
    small, large = vols
    torch.cuda.synchronize()
    n = min(small.state()["allocated"], capacity)
    if n < small.state()["allocated"]:
        # the pool overflowed: the table holds the same blocks as the small pool, by hand
        large.reset()
        for a in ("tsdf", "weight", "rgb_weight"):
            getattr(large, a)[:n * 512] = getattr(small, a)[:n * 512]
        large.rgb[:, :n * 512] = small.rgb[:, :n * 512]
        large.block_key[:n] = small.block_key[:n]
        large.state_t[0] = n
        keys = small.block_key[:n].cpu().numpy().view(np.uint64)
        tab, slots = large.keys.cpu().numpy().view(np.uint64).copy(), large.slots.cpu().numpy().copy()
        mask = np.uint64(large.n_buckets - 1)
        with np.errstate(over="ignore"):
            for i, k in enumerate(keys):
                x = (k ^ (k >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
                x = (x ^ (x >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
                s = (x ^ (x >> np.uint64(31))) & np.uint64(0xFFFFFFFF) & mask
                while tab[s] != np.uint64(0xFFFFFFFFFFFFFFFF):
                    s = (s + np.uint64(1)) & mask
                tab[s], slots[s] = k, i
        large.keys.copy_(torch.as_tensor(tab.view(np.int64)))
        large.slots.copy_(torch.as_tensor(slots))
    for skip in (True, False):
        outs = []
        for vol in (small, large):
            keep = vol.block_min
            if not skip:
                vol.block_min = None
            outs.append(P.hash_raycast(vol, [cam, near]))
            vol.block_min = keep
        torch.cuda.synchronize()
        hits = 0
        for (da, ca), (db, cb) in zip(*outs):
            np.testing.assert_array_equal(h(da), h(db))
            np.testing.assert_array_equal(h(ca), h(cb))
            hits += int((da > 0).sum())
        assert hits > 50
