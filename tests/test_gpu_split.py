"""Force passes that share a particle's cell rows among several lanes.

How many lanes follows from the particle count, so the sizes here lie on both
sides of every change: forces against the oracle's pair sums (1e-12 in units
of the RMS force for FP64, 1e-5 for FP32-mixed, the bars of the other parity
tests; counts bit for bit), list forces equal to the cell walk's and batched
results equal to single-system calls bit for bit."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm
import workloads

from gpu_util import F64, Ctx, dev, force_errors, gpu_forces, host

pytestmark = pytest.mark.gpu


def some(n, name="droplet"):
    """A system of n of the named workload's particles."""
    s = workloads.make(name)
    idx = workloads.sample_indices(s.n, n, seed=17)
    return dataclasses.replace(s, x=s.x[idx], y=s.y[idx], z=s.z[idx], vx=s.vx[idx], vy=s.vy[idx],
                               vz=s.vz[idx])


@pytest.mark.parametrize("prec", [dcm.DCM_FP64, dcm.DCM_FP32_MIXED])
@pytest.mark.parametrize("n", [1, 17, 255, 7999, 8000, 15999, 16000, 31999, 32000, 100000])
def test_step_forces(n, prec):
    print(f"[gpu] step forces n={n} prec={prec}", flush=True)
    s = some(n)
    x, y, z = dev(s.x), dev(s.y), dev(s.z)
    f = [torch.zeros(n, **F64) for _ in range(3)]
    v = [torch.zeros(n, **F64) for _ in range(3)]
    rc = torch.zeros(n, **F64)
    grid = dcm.make_grid(s.box, s.h)
    rule = dcm.make_rule(*s.rule)
    with Ctx() as ctx:
        dcm.dcm_step(ctx, x, y, z, *v, *f, s.box, dcm.make_lj(), rule, grid,
                     dcm.rc_grid_for(rule, grid), dt=0.005, nsteps=0, prec=prec, rc=rc)
        assert dcm.dcm_sync_status(ctx) in (dcm.DCM_OK, dcm.DCM_ERR_DEGENERATE)
    idx = workloads.sample_indices(n, 2000, seed=5)
    ref = oracle.forces(s.x, s.y, s.z, host(rc), s.box, idx=idx)
    R = np.stack([ref["fx"], ref["fy"], ref["fz"]], 1)
    F = np.stack([host(t) for t in f], 1)[idx]
    if not np.any(R):
        assert not np.any(F)
        return
    emax, erms = force_errors(F, R)
    tol = 1e-12 if prec == dcm.DCM_FP64 else 1e-5
    assert emax <= tol and erms <= tol, (emax, erms)


@pytest.mark.parametrize("prec", [dcm.DCM_FP64, dcm.DCM_FP32_MIXED])
@pytest.mark.parametrize("n", [1, 300, 7999, 8000, 31999, 32000, 99999, 100000])
def test_list_and_batch_equal_single_calls(n, prec):
    print(f"[gpu] list, batch and single call n={n} prec={prec}", flush=True)
    s = some(n)
    rc = workloads.uniform_cutoffs(n, 2.5, 8.0, seed=3)
    one = gpu_forces(s, rc, prec=prec, edge=1.5, rc_bound=8.0)
    ref = oracle.forces(s.x, s.y, s.z, rc, s.box, idx=workloads.sample_indices(n, 500, seed=6))
    np.testing.assert_array_equal(one["nnbr"][workloads.sample_indices(n, 500, seed=6)],
                                  ref["nnbr"])
    x, y, z, r = dev(s.x), dev(s.y), dev(s.z), dev(rc)
    d = dict(x=x, y=y, z=z, rc=r, box=s.box, cell_edge=1.5, rc_bound=8.0,
             **{k: torch.zeros(n, **F64) for k in ("fx", "fy", "fz")},
             nnbr=torch.zeros(n, dtype=torch.int32, device=x.device),
             energy=torch.zeros(1, **F64), virial=torch.zeros(6, **F64),
             npairs=torch.zeros(1, dtype=torch.uint64, device=x.device))
    flags = dcm.DCM_EV_ENERGY | dcm.DCM_EV_VIRIAL | dcm.DCM_EV_COUNTS
    with Ctx() as ctx:
        dcm.dcm_forces_batched(ctx, [d], dcm.make_lj(), prec=prec, ev_flags=flags)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    F = np.stack([host(d[k]) for k in ("fx", "fy", "fz")], 1)
    np.testing.assert_array_equal(F, one["F"])
    np.testing.assert_array_equal(host(d["nnbr"]), one["nnbr"])
    assert float(host(d["energy"])[0]) == one["E"]
    np.testing.assert_array_equal(host(d["virial"]), one["W"])
    if prec != dcm.DCM_FP64:
        return  # the list reads the FP64 records, the walk the compact ones
    f = [torch.zeros(n, **F64) for _ in range(3)]
    with Ctx() as ctx:
        dcm.dcm_build_cells(ctx, x, y, z, r, s.box, 1.5, prec, rc_bound=8.0)
        dcm.dcm_build_list(ctx, 0.2)
        dcm.dcm_forces_list(ctx, dcm.make_lj(), *f, prec=prec)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    np.testing.assert_array_equal(np.stack([host(t) for t in f], 1), one["F"])


# 500,000 particles: two lanes with cutoffs up to 5, four with up to 8 (and two
# at one particle fewer)
@pytest.mark.parametrize("n,bound", [(499999, 8.0), (500000, 5.0), (500000, 8.0)])
def test_half_a_million(n, bound):
    print(f"[gpu] cell walk and list n={n} cutoffs up to {bound}", flush=True)
    rng = np.random.default_rng(n)
    m, box = 80, (90.0, 90.0, 90.0)
    site = rng.permutation(m ** 3)[:n]
    p = (np.stack(np.unravel_index(site, (m, m, m)), 1) + 0.5) * (90.0 / m)
    p += rng.uniform(-0.1, 0.1, p.shape)
    x, y, z = (np.ascontiguousarray(p[:, a]) for a in range(3))
    rc = rng.uniform(2.5, bound, n)
    idx = workloads.sample_indices(n, 400, seed=6)
    ref = oracle.forces(x, y, z, rc, box, idx=idx)
    d = [dev(a) for a in (x, y, z, rc)]
    f, fl = ([torch.zeros(n, **F64) for _ in range(3)] for _ in range(2))
    nn = torch.zeros(n, dtype=torch.int32, device=d[0].device)
    with Ctx() as ctx:
        dcm.dcm_build_cells(ctx, *d, box, 1.5, dcm.DCM_FP64, rc_bound=bound)
        dcm.dcm_forces(ctx, dcm.make_lj(), *f, prec=dcm.DCM_FP64, ev_flags=dcm.DCM_EV_COUNTS,
                       nnbr=nn)
        dcm.dcm_build_list(ctx, 0.1)
        dcm.dcm_forces_list(ctx, dcm.make_lj(), *fl, prec=dcm.DCM_FP64)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    F = np.stack([host(t) for t in f], 1)
    np.testing.assert_array_equal(np.stack([host(t) for t in fl], 1), F)
    np.testing.assert_array_equal(host(nn)[idx], ref["nnbr"])
    R = np.stack([ref["fx"], ref["fy"], ref["fz"]], 1)
    assert max(force_errors(F[idx], R)) <= 1e-12
