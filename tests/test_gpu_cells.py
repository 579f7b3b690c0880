"""The cell build over the sizes at which its launches change.

Cells of one workgroup's scan and one more, extended rows scanned by one
workgroup and by many, tiles past the two-launch scan, cells past the ranked
size and past one LDS sort, no particle and one: cell starts equal to the
oracle's, counts bit for bit and forces within 1e-12 of the RMS force of the
oracle's sums.  The geometries follow each other in one context, there and
back, so that each build finds what another left in the scratch arrays; the
same systems in one batch must give the single calls' bits, replays included.
"""
import types

import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm

from gpu_util import DEV, F64, Ctx, dev, force_errors, host

pytestmark = pytest.mark.gpu

# cells per axis (edge 1 in a box of as many units unless given), particles
ONE_SCAN = ((32, 32, 16), 1.0, 9000)  # 16384 cells
TWO_SCANS = ((113, 29, 5), 1.0, 9000)  # 16385
ROWS = ((2, 254, 254), 1.0, 4000)  # 256 x 256 extended rows
MORE_ROWS = ((2, 254, 255), 1.0, 4000)
TOTALS = ((257, 256, 256), 1.0, 3000)  # past 4096 tiles of 4096 cells
PILED = ((3, 3, 3), 4.0, 1200)  # about 44 a cell
SORTED = ((1, 1, 1), 18.0, 4700)  # all in one cell, past one LDS sort
EMPTY = ((4, 4, 4), 1.0, 0)
SINGLE = ((4, 4, 4), 1.0, 1)


def system(case, seed):
    """n particles of a jittered lattice (no two within 0.8), edge, cutoffs."""
    nc, edge, n = case
    box = tuple(float(c) * edge for c in nc)
    rng = np.random.default_rng(seed)
    m = [max(int(L / 1.02), 1) for L in box]
    site = rng.choice(m[0] * m[1] * m[2], size=n, replace=False)
    ijk = np.stack(np.unravel_index(site, m), 1)
    p = (ijk + 0.5) * (np.array(box) / m) + rng.uniform(-0.1, 0.1, (n, 3))
    bound = min(2.0, *(0.45 * L for L in box))
    x, y, z = (np.ascontiguousarray(p[:, a]) for a in range(3))
    return types.SimpleNamespace(x=x, y=y, z=z, box=box, n=n, nc=nc, edge=edge, bound=bound,
                                 rc=rng.uniform(0.6, 1.0, n) * bound)


def single(ctx, s):
    x, y, z, rc = dev(s.x), dev(s.y), dev(s.z), dev(s.rc)
    f = [torch.zeros(s.n, **F64) for _ in range(3)]
    nn = torch.zeros(s.n, dtype=torch.int32, device=DEV)
    start = torch.zeros(int(np.prod(s.nc)) + 1, dtype=torch.int32, device=DEV)
    dcm.dcm_build_cells(ctx, x, y, z, rc, s.box, s.edge, dcm.DCM_FP64, cell_start=start,
                        rc_bound=s.bound)
    dcm.dcm_forces(ctx, dcm.make_lj(), *f, prec=dcm.DCM_FP64, ev_flags=dcm.DCM_EV_COUNTS, nnbr=nn)
    assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    assert dcm.dcm_cell_dims(ctx)[0] == list(s.nc)
    return np.stack([host(t) for t in f], 1), host(nn), host(start)


@pytest.mark.parametrize("cases", [(ONE_SCAN, TWO_SCANS), (ROWS, MORE_ROWS), (TOTALS, SINGLE),
                                   (PILED, SORTED), (EMPTY, SINGLE, PILED), (SORTED, ONE_SCAN)])
def test_builds_in_turn_and_batched(cases):
    systems = [system(c, 11 + k) for k, c in enumerate(cases)]
    got = {}
    with Ctx() as ctx:
        for k in list(range(len(cases))) + list(range(len(cases)))[::-1]:
            s = systems[k]
            print(f"[gpu] cells {s.nc} edge {s.edge} n={s.n}", flush=True)
            F, nn, start = single(ctx, s)
            if k in got:
                np.testing.assert_array_equal(F, got[k][0])
                np.testing.assert_array_equal(nn, got[k][1])
                np.testing.assert_array_equal(start, got[k][2])
                continue
            got[k] = (F, nn, start)
            np.testing.assert_array_equal(start, oracle.cells(s.x, s.y, s.z, s.box, s.nc)[1])
            if s.n == 0:
                continue
            ref = oracle.forces(s.x, s.y, s.z, s.rc, s.box)
            np.testing.assert_array_equal(nn, ref["nnbr"])
            R = np.stack([ref["fx"], ref["fy"], ref["fz"]], 1)
            if np.any(R):
                assert max(force_errors(F, R)) <= 1e-12
            else:
                assert not np.any(F)
    batch = [dict(x=dev(s.x), y=dev(s.y), z=dev(s.z), rc=dev(s.rc), box=s.box, cell_edge=s.edge,
                  rc_bound=s.bound, nnbr=torch.zeros(s.n, dtype=torch.int32, device=DEV),
                  **{k: torch.zeros(s.n, **F64) for k in ("fx", "fy", "fz")}) for s in systems]
    print("[gpu] the same systems in one batch, four calls", flush=True)
    with Ctx() as ctx:
        arr = batch
        for _ in range(4):  # the last ones replay the recorded graph
            arr = dcm.dcm_forces_batched(ctx, arr, dcm.make_lj(), prec=dcm.DCM_FP64,
                                         ev_flags=dcm.DCM_EV_COUNTS, use_graph=True)
            assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK, dcm.dcm_last_error(ctx)
            for k, d in enumerate(batch):
                F = np.stack([host(d[c]) for c in ("fx", "fy", "fz")], 1)
                np.testing.assert_array_equal(F, got[k][0])
                np.testing.assert_array_equal(host(d["nnbr"]), got[k][1])
                for c in ("fx", "fy", "fz", "nnbr"):
                    d[c].zero_()
