"""The majority vote over grids at which its launches change.

Rows of one voxel (a launch per pass), of part of a word, of whole words and
one voxel more, and the widest rows kept in LDS and one voxel more; row counts
below, at and past a tile, and many tiles.  Uniform noise, so that regions grow through all passes: threshold,
phase map and interface equal the oracle's."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm

from gpu_util import DEV, Ctx, dev, host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nv", [(1, 20, 20), (2, 9, 17), (31, 8, 8), (32, 16, 7), (33, 1, 40),
                                (100, 17, 33), (224, 25, 9), (225, 3, 24), (384, 10, 12),
                                (385, 10, 12), (20, 180, 170), (70, 177, 190)])
def test_noise_matches_oracle(nv):
    print(f"[gpu] majority vote on {nv} voxels", flush=True)
    box = tuple(float(v) for v in nv)
    rng = np.random.default_rng(sum(nv))
    n = int(0.4 * np.prod(nv)) + 20
    x, y, z = (rng.uniform(0.0, L, n) for L in box)
    ref = oracle.detect_interface(x, y, z, box, 1.0, split=11.0)
    grid = dcm.make_grid(box, 1.0)
    assert tuple(grid.n) == nv
    seg = torch.zeros(int(np.prod(nv)), dtype=torch.uint8, device=DEV)
    iface = torch.zeros_like(seg)
    thr = torch.zeros(1, dtype=torch.int32, device=DEV)
    args = [dev(c) for c in (x, y, z)]
    with Ctx() as ctx:
        for call in (dcm.dcm_detect_interface, dcm.dcm_detect_interface_noalloc):
            call(ctx, *args, box, grid, seg, iface, split=11.0, threshold_out=thr)
            assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
            assert int(host(thr)[0]) == ref["threshold"]
            np.testing.assert_array_equal(host(seg), ref["seg"])
            np.testing.assert_array_equal(host(iface), ref["iface"])
            seg.zero_()
            iface.zero_()
