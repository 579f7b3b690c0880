"""Detection and a whole step on grids of every number of planes per workgroup (4,
8, 16, 32), with particles that do not overlap, so that the device's status is
known: DCM_ERR_DEGENERATE where the oracle finds a single phase, else DCM_OK --
no sweep left unconverged, no cutoff out of range, no ghost overflow.  Counts,
threshold, phase map, interface and cutoffs against the oracle (cutoffs 1e-12 of
rc_max), forces of the step against its pair sums (1e-12 of the RMS force)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm
import workloads

from gpu_util import DEV, F64, Ctx, dev, force_errors, host

pytestmark = pytest.mark.gpu

RULE = (2.5, 6.0, 4.0)


def particles(nv, kind):
    """Jittered lattice sites: a ball of liquid across the periodic faces and a
    thin vapour, or one phase throughout."""
    rng = np.random.default_rng(sum(nv))
    box = np.array(nv, float)
    m = np.floor(box / 1.08).astype(int)
    site = np.stack(np.meshgrid(*(np.arange(k) for k in m), indexing="ij"), -1).reshape(-1, 3)
    p = (site + 0.5) * (box / m)
    if kind == "ball":
        d = np.minimum(p, box - p)
        p = p[(np.linalg.norm(d, axis=1) < 0.45 * min(nv)) | (rng.uniform(0, 1, len(p)) < 0.03)]
    p = (p + rng.uniform(-0.05, 0.05, p.shape)) % box
    return tuple(float(k) for k in nv), [np.ascontiguousarray(p[:, a]) for a in range(3)]


@pytest.mark.parametrize("nv,kind", [((18, 13, 37), "ball"), ((31, 13, 65), "ball"),
                                     ((32, 13, 100), "ball"), ((33, 60, 90), "ball"),
                                     ((64, 90, 181), "ball"), ((65, 64, 80), "ball"),
                                     ((100, 80, 200), "ball"), ((130, 100, 200), "ball"),
                                     ((18, 13, 37), "liquid"), ((64, 60, 80), "liquid")])
def test_status(nv, kind):
    print(f"[gpu] detection status on {nv} voxels, {kind}", flush=True)
    box, x = particles(nv, kind)
    n = len(x[0])
    ref = oracle.pipeline(*x, box, 1.0, RULE, idx=[0])
    assert ref["degenerate"] == (kind == "liquid")
    want = dcm.DCM_ERR_DEGENERATE if ref["degenerate"] else dcm.DCM_OK
    nvox = int(np.prod(nv))
    grid, rule = dcm.make_grid(box, 1.0), dcm.make_rule(*RULE)
    counts = torch.zeros(nvox, dtype=torch.uint32, device=DEV)
    seg = torch.zeros(nvox, dtype=torch.uint8, device=DEV)
    iface = torch.zeros_like(seg)
    thr = torch.zeros(1, dtype=torch.int32, device=DEV)
    d = [dev(a) for a in x]
    f, v = ([torch.zeros(n, **F64) for _ in range(3)] for _ in range(2))
    rc = torch.zeros(n, **F64)
    with Ctx() as ctx:
        dcm.dcm_detect_interface(ctx, *d, box, grid, seg, iface, counts=counts, threshold_out=thr)
        assert dcm.dcm_sync_status(ctx) == want
        dcm.dcm_step(ctx, *d, *v, *f, box, dcm.make_lj(), rule, grid,
                     dcm.rc_grid_for(rule, grid), dt=0.005, nsteps=0, rc=rc)
        assert dcm.dcm_sync_status(ctx) == want
    np.testing.assert_array_equal(host(counts), ref["counts"])
    np.testing.assert_array_equal(host(seg), ref["seg"])
    np.testing.assert_array_equal(host(iface), ref["iface"])
    if not ref["degenerate"]:
        assert int(host(thr)[0]) == ref["threshold"]
    assert np.max(np.abs(host(rc) - ref["rc"])) <= 1e-12 * RULE[1]
    idx = workloads.sample_indices(n, 300, seed=5)
    fr = oracle.forces(*x, host(rc), box, idx=idx)
    R = np.stack([fr["fx"], fr["fy"], fr["fz"]], 1)
    F = np.stack([host(t) for t in f], 1)[idx]
    assert max(force_errors(F, R)) <= 1e-12
