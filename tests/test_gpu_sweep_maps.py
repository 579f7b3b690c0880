"""dcm_sweep_distance on maps whose interface is not that of the phase map: every
low-density voxel and every marked voxel is a source, wherever the marks are.
Grids of one tile and of many.  And long thin grids, of more than 65,535 layers of
tiles.  Against the oracle's distances: 1e-12 of rc_grid, the bar of the other
sweep tests."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm

from gpu_util import F64, Ctx, dev, host

pytestmark = pytest.mark.gpu


def maps(kind, nv):
    rng = np.random.default_rng(int(np.prod(nv)))
    nx, ny, nz = nv
    z, y, x = np.meshgrid(*(np.arange(k) for k in nv[::-1]), indexing="ij")
    r = np.sqrt((x - 0.4 * nx) ** 2 + (y - 0.5 * ny) ** 2 + (z - 0.55 * nz) ** 2)
    seg = (r < 0.4 * min(nv)).astype(np.uint8)
    marked = np.zeros_like(seg)
    if kind == "few marks":  # in one corner of the vapour only
        marked[:2, :2, :2] = 1
    elif kind == "marks inside":  # a few liquid voxels, as sources of their own
        seg[:] = 1
        marked[rng.uniform(0, 1, seg.shape) < 3.0 / seg.size] = 1
        marked[nz // 2, ny // 2, nx // 2] = 1
    elif kind == "vapour side":  # the vapour voxels next to the liquid
        near = np.zeros_like(seg)
        for axis in range(3):
            for step in (1, -1):
                near |= np.roll(seg, step, axis)
        marked = near & (1 - seg)
    elif kind == "one vapour voxel":  # where eight tiles meet
        seg[:] = 1
        seg[8 % nz, 8 % ny, 16 % nx] = 0
    return seg.ravel(), marked.ravel()


@pytest.mark.parametrize("nv", [(16, 8, 8), (18, 10, 10), (50, 33, 41), (96, 64, 72)])
@pytest.mark.parametrize("kind", ["no marks", "few marks", "marks inside", "vapour side",
                                  "one vapour voxel"])
def test_any_marks(kind, nv):
    print(f"[gpu] sweep of {kind} on {nv}", flush=True)
    seg, marked = maps(kind, nv)
    rcg = 12.0
    D, passes = oracle.fsm(nv, (1.0, 1.0, 1.0), seg, marked, rcg)
    assert passes > 0
    grid = dcm.make_grid(tuple(float(k) for k in nv), 1.0)
    dist = torch.zeros(seg.size, **F64)
    with Ctx() as ctx:
        dcm.dcm_sweep_distance(ctx, dev(seg, torch.uint8), dev(marked, torch.uint8), grid, rcg,
                               500, dist)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    assert np.max(np.abs(host(dist) - D)) <= 1e-12 * rcg


@pytest.mark.parametrize("nv", [(2, 3, 600000), (3, 1, 530000)])
def test_long_thin_grid(nv):
    print(f"[gpu] sweep of a long thin grid {nv}", flush=True)
    rng = np.random.default_rng(3)
    n = int(np.prod(nv))
    seg = (rng.uniform(0, 1, n) > 0.02).astype(np.uint8)
    marked = oracle.interface(nv, seg)
    D, passes = oracle.fsm(nv, (1.0, 1.0, 1.0), seg, marked, 8.0)
    assert passes > 0
    grid = dcm.make_grid(tuple(float(k) for k in nv), 1.0)
    dist = torch.zeros(n, **F64)
    with Ctx() as ctx:
        dcm.dcm_sweep_distance(ctx, dev(seg, torch.uint8), dev(marked, torch.uint8), grid, 8.0,
                               500, dist)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    assert np.max(np.abs(host(dist) - D)) <= 8e-12
