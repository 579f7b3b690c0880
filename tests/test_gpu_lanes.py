"""Forces on both sides of every change of the lanes that share a particle's
rows, where the change follows n (6 / rc_max)^3, the spread of the cutoffs or the
pair rule: dcm_step's own passes, and the symmetric rule at many particles.  Against the oracle's pair
sums (1e-12 in units of the RMS force for FP64, 1e-5 for FP32-mixed, the bars of
the other parity tests)."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm
import workloads

from gpu_util import F64, Ctx, dev, force_errors, host

pytestmark = pytest.mark.gpu

BAR = {dcm.DCM_FP64: 1e-12, dcm.DCM_FP32_MIXED: 1e-5}


def slab(n):
    """n jittered lattice sites: a dense slab across z and a thin vapour."""
    rng = np.random.default_rng(n)
    m = (int(np.ceil((n / 1.6) ** (1.0 / 3.0))),) * 2
    m += (-(-16 * n // (10 * m[0] * m[1])) * 2,)
    a = 1.1  # 0.75 particles per unit volume in the slab
    box = tuple(k * a for k in m)
    site = np.stack(np.unravel_index(np.arange(np.prod(m)), m), 1)
    order = np.argsort(np.abs(site[:, 2] - m[2] / 2.0) + rng.uniform(0, 1e-3, len(site)))
    liquid = int(0.97 * n)
    pick = np.concatenate([order[:liquid], rng.permutation(order[liquid:])[:n - liquid]])
    p = (site[rng.permutation(pick)] + 0.5) * a + rng.uniform(-0.1, 0.1, (n, 3))
    return box, [np.ascontiguousarray(p[:, k]) for k in range(3)]


def check(F, x, rc, box, rule, prec):
    idx = workloads.sample_indices(len(rc), 400, seed=5)
    ref = oracle.forces(*x, rc, box, rule=rule, idx=idx)
    R = np.stack([ref["fx"], ref["fy"], ref["fz"]], 1)
    emax, erms = force_errors(F[idx], R)
    assert emax <= BAR[prec] and erms <= BAR[prec], (emax, erms)


# n (6 / 3)^3 = 8 n: 16, 8, 4, 2 lanes and one from 2000, 18750, 37500 and
# 375000 on (compact records); 16, 8 and 4 from 2500 and 18750 on (FP64)
OWN = [(dcm.DCM_FP32_MIXED, n, 2.5, 3.0)
       for n in (1999, 2000, 18749, 18750, 37499, 37500, 374999, 375000)]
OWN += [(dcm.DCM_FP64, n, 2.5, 3.0) for n in (2499, 2500, 18749, 18750)]
# from 500,000 particles on one lane if all cutoffs exceed 0.6 rc_max (two and,
# in FP64, four before); else four in FP64 below 450,000 / (6 / rc_max)^3, then two
OWN += [(p, n, 2.5, 4.0) for p in (dcm.DCM_FP64, dcm.DCM_FP32_MIXED) for n in (499999, 500000)]
OWN += [(dcm.DCM_FP64, 500000, 2.5, r) for r in (6.0, 6.4)]


@pytest.mark.parametrize("prec,n,rc_min,rc_max", OWN)
def test_step(prec, n, rc_min, rc_max):
    print(f"[gpu] step forces n={n} prec={prec} {rc_min}-{rc_max}", flush=True)
    box, x = slab(n)
    d = [dev(a) for a in x]
    f, v = ([torch.zeros(n, **F64) for _ in range(3)] for _ in range(2))
    rc = torch.zeros(n, **F64)
    grid, rule = dcm.make_grid(box, 1.0), dcm.make_rule(rc_min, rc_max, 5.0)
    with Ctx() as ctx:
        dcm.dcm_step(ctx, *d, *v, *f, box, dcm.make_lj(), rule, grid, dcm.rc_grid_for(rule, grid),
                     dt=0.005, nsteps=0, prec=prec, rc=rc)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    rc = host(rc)
    assert rc.min() < rc_min + 0.2 and rc.max() == rc_max
    check(np.stack([host(t) for t in f], 1), x, rc, box, dcm.DCM_PAIR_OWN, prec)


# two lanes up to 349,999 particles, then one; in a batch too, bit for bit
@pytest.mark.parametrize("prec", [dcm.DCM_FP64, dcm.DCM_FP32_MIXED])
@pytest.mark.parametrize("n", [349999, 350000])
def test_symmetric_rule(n, prec):
    print(f"[gpu] symmetric rule n={n} prec={prec}", flush=True)
    box, x = slab(n)
    rc = workloads.uniform_cutoffs(n, 2.5, 3.0, seed=3)
    d, r = [dev(a) for a in x], dev(rc)
    f, fb = ([torch.zeros(n, **F64) for _ in range(3)] for _ in range(2))
    s = dict(zip(("x", "y", "z", "fx", "fy", "fz"), d + fb), rc=r, box=box, cell_edge=1.5,
             rc_bound=3.0)
    with Ctx() as ctx:
        dcm.dcm_build_cells(ctx, *d, r, box, 1.5, prec, rc_bound=3.0)
        dcm.dcm_forces(ctx, dcm.make_lj(), *f, pair_rule=dcm.DCM_PAIR_MAX, prec=prec)
        dcm.dcm_forces_batched(ctx, [s], dcm.make_lj(), pair_rule=dcm.DCM_PAIR_MAX, prec=prec)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    F = np.stack([host(t) for t in f], 1)
    np.testing.assert_array_equal(np.stack([host(t) for t in fb], 1), F)
    check(F, x, rc, box, dcm.DCM_PAIR_MAX, prec)
