"""Sweeps whose passes outlast the launches of their own, so that one launch
goes on with the rest, its workgroups taking the tiles of each pass in turn:
tens of tiles active that late, and a grid of few tiles, where that launch begins
early.  Against the oracle's distances (the fixed point of the same update in
another order): 1e-12 of rc_grid, the bar of the other sweep tests; the same bits
on every run; and the passes counted exactly."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm

from gpu_util import DEV, F64, Ctx, dev, host

pytestmark = pytest.mark.gpu


def cylinders(nv, d, seed):
    """Liquid cylinders along x, one per d x d columns, rough at one end only: the
    corrections that the rough ends make creep along the axes, tile by tile."""
    rng = np.random.default_rng(seed)
    z, y, x = np.meshgrid(*(np.arange(k) for k in nv[::-1]), indexing="ij")
    r = np.hypot(y % d - d / 2.0 + 0.3, z % d - d / 2.0 + 0.2)
    edge = 0.4 * d + np.where(x < 12, rng.integers(-2, 3, x.shape), 0)
    return (r < edge).astype(np.uint8).ravel()


def gyroid(nv, period):
    z, y, x = np.meshgrid(*(np.arange(k) * (2.0 * np.pi / period) for k in nv[::-1]),
                          indexing="ij")
    g = np.sin(x) * np.cos(y) + np.sin(y) * np.cos(z) + np.sin(z) * np.cos(x)
    return (g > -0.8).astype(np.uint8).ravel()


# (voxels, spacing, map, rc_grid, least passes)
CASES = [
    ((480, 36, 144), (1.0, 1.0, 1.0), "cylinders", 8.0, 24),
    ((480, 36, 144), (0.9, 1.1, 1.05), "cylinders", 8.0, 24),
    ((480, 72, 36), (0.5, 0.5, 0.5), "cylinders", 4.0, 24),
    ((64, 16, 16), (1.0, 1.0, 1.0), "gyroid", 20.0, 8),
    ((61, 13, 19), (1.0, 0.9, 0.8), "gyroid", 20.0, 8),
]


@pytest.mark.parametrize("nv,hv,kind,rcg,least", CASES)
def test_passes_past_their_own_launches(nv, hv, kind, rcg, least):
    print(f"[gpu] sweep tail {nv} {hv} {kind}", flush=True)
    seg = cylinders(nv, 36, 5) if kind == "cylinders" else gyroid(nv, 64)
    iface = oracle.interface(nv, seg)
    D, passes = oracle.fsm(nv, hv, seg, iface, rcg)
    assert passes > 0
    grid = dcm.make_grid([n * h for n, h in zip(nv, hv)], 1.0)
    for a in range(3):
        grid.n[a], grid.h[a] = nv[a], hv[a]
    s, f = dev(seg, torch.uint8), dev(iface, torch.uint8)
    dist, again = torch.zeros(seg.size, **F64), torch.zeros(seg.size, **F64)
    waves, waves2 = (torch.zeros(1, dtype=torch.int32, device=DEV) for _ in range(2))
    with Ctx() as ctx:
        dcm.dcm_sweep_distance(ctx, s, f, grid, rcg, 500, dist, waves_out=waves)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        n = int(host(waves)[0])
        print(f"[gpu]   {n} passes", flush=True)
        assert n >= least
        assert np.max(np.abs(host(dist) - D)) <= 1e-12 * rcg
        for limit in (500, 60, n + 1, n):
            dcm.dcm_sweep_distance(ctx, s, f, grid, rcg, limit, again, waves_out=waves2)
            assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
            assert int(host(waves2)[0]) == n
            np.testing.assert_array_equal(host(again), host(dist))
        dcm.dcm_sweep_distance(ctx, s, f, grid, rcg, n - 1, again)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_ERR_NOT_CONVERGED
