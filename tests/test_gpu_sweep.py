"""The tiled distance sweep where its tiles, halos and lists can go wrong:
grids thinner than a tile or one voxel past it, unequal voxel edges, and a
sweep that needs more passes than get launches of their own.  Against the
oracle's distances (the fixed point of the same update in another order):
1e-12 of rc_grid, the bar of the other sweep tests."""

import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm
import workloads

from gpu_util import DEV, F64, Ctx, dev, host

pytestmark = pytest.mark.gpu


def bounded(a, b, scale):
    assert np.max(np.abs(a - b)) <= 1e-12 * scale


@pytest.mark.parametrize("box", [(5.0, 6.0, 33.0), (16.0, 8.0, 40.0), (17.0, 9.0, 41.0),
                                 (18.0, 10.0, 42.0), (33.0, 12.0, 64.0), (13.4, 13.4, 60.0),
                                 (34.5, 17.3, 49.2)])
def test_step_distances(box):
    """dcm_step's distances at the particles (its sweep takes tiles on every grid)."""
    print(f"[gpu] step distances {box}", flush=True)
    rc_max = 0.49 * min(box)
    s = workloads.slab("s", box, box[2] / 3.0, box[2] / 3.0, seed=11,
                       rule=(min(2.0, 0.9 * rc_max), rc_max, 5.0))
    ref = oracle.pipeline(s.x, s.y, s.z, s.box, s.h, s.rule, idx=[0])
    f = [torch.zeros(s.n, **F64) for _ in range(3)]
    v = [torch.zeros(s.n, **F64) for _ in range(3)]
    delta = torch.zeros(s.n, **F64)
    grid = dcm.make_grid(s.box, s.h)
    rule = dcm.make_rule(*s.rule)
    rcg = dcm.rc_grid_for(rule, grid)
    with Ctx() as ctx:
        dcm.dcm_step(ctx, dev(s.x), dev(s.y), dev(s.z), *v, *f, s.box, dcm.make_lj(), rule, grid,
                     rcg, dt=0.005, nsteps=0, delta=delta)
        assert dcm.dcm_sync_status(ctx) == (dcm.DCM_ERR_DEGENERATE if ref["degenerate"]
                                            else dcm.DCM_OK)
    bounded(host(delta), ref["delta"], rcg)


@pytest.mark.parametrize("nv", [(18, 10, 10), (160, 36, 36), (480, 36, 36)])
@pytest.mark.parametrize("hv", [(1.0, 1.0, 1.0), (0.9, 1.1, 1.05)])
def test_sweep_along_a_cylinder(nv, hv):
    """A liquid cylinder along x, rough at one end only: the corrections that
    the rough end makes creep along the axis, tile by tile."""
    print(f"[gpu] cylinder sweep {nv} {hv}", flush=True)
    rng = np.random.default_rng(5)
    z, y, x = np.meshgrid(*(np.arange(k) for k in nv[::-1]), indexing="ij")
    r = np.hypot(y - nv[1] / 2.0 + 0.3, z - nv[2] / 2.0 + 0.2)
    edge = 0.4 * nv[1] + np.where(x < 12, rng.integers(-2, 3, x.shape), 0)
    seg = (r < edge).astype(np.uint8).ravel()
    iface = oracle.interface(nv, seg)
    rcg = 8.0
    D, passes = oracle.fsm(nv, hv, seg, iface, rcg)
    assert passes > 0
    grid = dcm.make_grid([n * h for n, h in zip(nv, hv)], 1.0)
    for a in range(3):
        grid.n[a], grid.h[a] = nv[a], hv[a]
    dist = torch.zeros(seg.size, **F64)
    waves = torch.zeros(1, dtype=torch.int32, device=DEV)
    with Ctx() as ctx:
        dcm.dcm_sweep_distance(ctx, dev(seg, torch.uint8), dev(iface, torch.uint8), grid, rcg, 500,
                               dist, waves_out=waves)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        print(f"[gpu]   {int(host(waves)[0])} passes", flush=True)
        bounded(host(dist), D, rcg)
        # the same with just as many passes as it took, and one too few
        dist2 = torch.zeros_like(dist)
        n = int(host(waves)[0])
        dcm.dcm_sweep_distance(ctx, dev(seg, torch.uint8), dev(iface, torch.uint8), grid, rcg, n,
                               dist2)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        np.testing.assert_array_equal(host(dist2), host(dist))
        if n > 2:
            dcm.dcm_sweep_distance(ctx, dev(seg, torch.uint8), dev(iface, torch.uint8), grid, rcg,
                                   n - 1, dist2)
            assert dcm.dcm_sync_status(ctx) == dcm.DCM_ERR_NOT_CONVERGED


# tiles of the first pass searched by the workgroups (256, 4352) and listed
# beforehand (320, 512, 4096)
@pytest.mark.parametrize("nv", [(64, 64, 64), (65, 64, 64), (128, 64, 64), (256, 128, 128),
                                (257, 128, 128)])
def test_first_pass_of_a_ball(nv):
    print(f"[gpu] ball sweep {nv}", flush=True)
    z, y, x = np.meshgrid(*(np.arange(k, dtype=np.float32) for k in nv[::-1]), indexing="ij")
    r = np.sqrt((x - 20.3) ** 2 + (y - nv[1] / 2.0 + 0.3) ** 2 + (z - nv[2] / 2.0) ** 2)
    seg = (r < 0.3 * nv[1]).astype(np.uint8).ravel()
    iface = oracle.interface(nv, seg)
    rcg = 8.0
    D, _ = oracle.fsm(nv, (1.0, 1.0, 1.0), seg, iface, rcg)
    grid = dcm.make_grid(tuple(float(k) for k in nv), 1.0)
    dist = torch.zeros(int(np.prod(nv)), **F64)
    with Ctx() as ctx:
        dcm.dcm_sweep_distance(ctx, dev(seg, torch.uint8), dev(iface, torch.uint8), grid, rcg, 200,
                               dist)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    bounded(host(dist), D, rcg)
