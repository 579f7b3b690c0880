"""The gray values, the split and the sweep's sources on grids of every number
of planes per workgroup (4, 8, 16, 32) and of rows of one word, two, a part of a
third: counts, threshold, phase map and interface equal the oracle's, and
dcm_step's cutoffs, whose sources come from the bit-packed map, those of the
separate calls to 1e-12 of rc_max."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm

from gpu_util import DEV, F64, Ctx, dev, host

pytestmark = pytest.mark.gpu

RULE = (2.5, 6.0, 4.0)


@pytest.mark.parametrize("nv", [(18, 13, 37), (31, 13, 65), (32, 13, 100), (33, 60, 90),
                                (64, 90, 181), (65, 64, 80), (100, 80, 200), (130, 100, 200)])
def test_detection_and_cutoffs(nv):
    print(f"[gpu] detection on {nv} voxels", flush=True)
    box = tuple(float(v) for v in nv)
    rng = np.random.default_rng(sum(nv))
    # a liquid ball (across the periodic faces) and gas
    n = int(0.5 * np.prod(nv))
    p = rng.uniform(0.0, 1.0, (n, 3)) * box
    d = np.minimum(p, box - p)
    keep = (np.linalg.norm(d, axis=1) < 0.45 * min(nv) + 4.0) | (rng.uniform(0, 1, n) < 0.04)
    x, y, z = (np.ascontiguousarray(p[keep, a]) for a in range(3))
    n = len(x)
    ref = oracle.detect_interface(x, y, z, box, 1.0)
    nvox = int(np.prod(nv))
    grid, rule = dcm.make_grid(box, 1.0), dcm.make_rule(*RULE)
    counts = torch.zeros(nvox, dtype=torch.uint32, device=DEV)
    seg = torch.zeros(nvox, dtype=torch.uint8, device=DEV)
    iface = torch.zeros_like(seg)
    thr = torch.zeros(1, dtype=torch.int32, device=DEV)
    dist = torch.zeros(nvox, **F64)
    rc, rc_step, delta = (torch.zeros(n, **F64) for _ in range(3))
    args = [dev(c) for c in (x, y, z)]
    rc_grid = dcm.dcm_rc_grid(rule, grid)
    ok = (dcm.DCM_OK, dcm.DCM_ERR_DEGENERATE)
    with Ctx() as ctx:
        dcm.dcm_detect_interface(ctx, *args, box, grid, seg, iface, counts=counts,
                                 threshold_out=thr)
        dcm.dcm_sweep_distance(ctx, seg, iface, grid, rc_grid, 200, dist)
        dcm.dcm_assign_cutoffs(ctx, *args, box, grid, dist, rule, rc, delta)
        assert dcm.dcm_sync_status(ctx) in ok
        np.testing.assert_array_equal(host(counts), ref["counts"])
        assert int(host(thr)[0]) == ref["threshold"]
        np.testing.assert_array_equal(host(seg), ref["seg"])
        np.testing.assert_array_equal(host(iface), ref["iface"])
        zero = [torch.zeros(n, **F64) for _ in range(6)]
        dcm.dcm_step(ctx, *args, *zero, box, dcm.make_lj(), rule, grid, rc_grid, dt=0.0,
                     nsteps=0, prec=dcm.DCM_FP64, rc=rc_step)
        dcm.dcm_sync_status(ctx)  # (overlapping particles: forces may not be finite)
    assert np.max(np.abs(host(rc_step) - host(rc))) <= 1e-12 * RULE[1]
    assert host(rc).min() < RULE[1]
