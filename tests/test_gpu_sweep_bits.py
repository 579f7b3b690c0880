"""The distance update's square root and quotient, bit for bit: synchronous waves
on a grid thinner than a tile against the same waves in numpy, whose square root
and quotient are correctly rounded.  Random maps and spacings, of every size that
spacings are taken at and far beyond."""
import numpy as np
import pytest
import torch

import oracle
import paper_1701_05242_amd as dcm

from gpu_util import F64, Ctx, dev, host

pytestmark = pytest.mark.gpu


def update(a, h):
    """The Godunov update from the smaller face neighbours a[3] (spacings h[3])."""
    w = 1.0 / (h * h)
    k = np.argsort(a, axis=0, kind="stable")
    a = np.take_along_axis(a, k, 0)
    hk, wk = h[k], w[k]
    with np.errstate(invalid="ignore", over="ignore"):
        d1 = a[0] + hk[0]
        b1, b2 = a[1] - a[0], a[2] - a[0]
        p1, p2 = wk[1] * b1, wk[2] * b2
        A = wk[0] + wk[1]
        disc = np.maximum(p1 * p1 - A * (p1 * b1 - 1.0), 0.0)
        d2 = a[0] + (p1 + np.sqrt(disc)) / A
        A, B = A + wk[2], p1 + p2
        disc = np.maximum(B * B - A * ((p1 * b1 + p2 * b2) - 1.0), 0.0)
        d3 = a[0] + (B + np.sqrt(disc)) / A
    d = np.where(d1 <= a[1], d1, np.where(d2 <= a[2], d2, d3))
    return np.where(np.isinf(a[0]), a[0], d)


def waves(source, h, limit):
    D = np.where(source, 0.0, np.inf)
    for n in range(1, 200):
        a = np.stack([np.minimum(np.roll(D, 1, ax), np.roll(D, -1, ax)) for ax in (2, 1, 0)])
        v = update(a, h)
        new = np.where(~source & (v < D) & (v <= limit), v, D)
        if np.array_equal(new, D):
            return np.minimum(D, limit), n
        D = new
    raise AssertionError("no end")


@pytest.mark.parametrize("scale", [1.0, 0.37, 1e-3, 1e3, 1e-100, 1e100])
@pytest.mark.parametrize("equal", [True, False])
def test_waves_bit_for_bit(scale, equal):
    print(f"[gpu] waves bit for bit, spacings of {scale}, equal={equal}", flush=True)
    rng = np.random.default_rng(int(abs(np.log(scale)) * 10) + equal)
    nv = (17, 9, 40)
    with Ctx() as ctx:
        for trial in range(12):
            h = scale * (np.full(3, rng.uniform(0.5, 1.5)) if equal else rng.uniform(0.5, 1.5, 3))
            p = (0.002, 0.01, 0.05, 0.2)[trial % 4]
            seg = (rng.uniform(0, 1, nv[::-1]) > p).astype(np.uint8)
            marked = oracle.interface(nv, seg.ravel()) if trial % 2 else np.zeros(seg.size, np.uint8)
            source = (seg == 0) | (marked.reshape(seg.shape) != 0)
            limit = 7.3 * float(h.max())
            want, n = waves(source, h, limit)
            grid = dcm.make_grid(tuple(float(k) for k in nv), 1.0)
            for a in range(3):
                grid.n[a], grid.h[a] = nv[a], float(h[a])
            dist = torch.zeros(seg.size, **F64)
            count = torch.zeros(1, dtype=torch.int32, device=dist.device)
            dcm.dcm_sweep_distance(ctx, dev(seg.ravel(), torch.uint8), dev(marked, torch.uint8),
                                   grid, limit, 300, dist, waves_out=count)
            assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
            assert int(host(count)[0]) == n
            np.testing.assert_array_equal(host(dist), want.ravel())
