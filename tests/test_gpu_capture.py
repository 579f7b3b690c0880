"""Library calls around stream capture.  The cells' counters are right whatever a
capture left behind: a capture that is dropped, or fails, after it made the
buffers grow leaves the next eager build a buffer nothing has cleared; a captured
build is replayed between eager builds.  One plan serves a batch's calls of any
rule and precision, and scratch is sized for all of them, so a call can be
captured after one of another kind.  Forces and counts equal those of a fresh
context bit for bit."""
import ctypes

import numpy as np
import pytest
import torch

import paper_1701_05242_amd as dcm
import workloads

from gpu_util import DEV, F64, dev, host

pytestmark = pytest.mark.gpu

RELAXED = 2  # hipStreamCaptureModeRelaxed
EDGE, BOUND = 1.5, 6.0


def hip(name, *args):
    # the runtime the library is linked with
    return getattr(dcm.load_library(), name)(*args)


def handle(stream):
    return ctypes.c_void_p(stream.cuda_stream)


def begin(stream):
    assert hip("hipStreamBeginCapture", handle(stream), ctypes.c_int(RELAXED)) == 0


def end(stream):
    g = ctypes.c_void_p()
    code = hip("hipStreamEndCapture", handle(stream), ctypes.byref(g))
    hip("hipGetLastError")
    return code, g


def poison(nbytes):
    """Device memory of every size up to nbytes that holds no zeros, given back."""
    keep = []
    while nbytes >= 4096:
        keep.append(torch.full((nbytes // 4,), 0x01010101, dtype=torch.int32, device=DEV))
        nbytes //= 2
    torch.cuda.synchronize()
    del keep
    torch.cuda.empty_cache()


def system(n, seed):
    rng = np.random.default_rng(seed)
    m, L = 24, 27.0
    site = rng.permutation(m ** 3)[:n]
    p = (np.stack(np.unravel_index(site, (m, m, m)), 1) + 0.5) * (L / m)
    p += rng.uniform(-0.05, 0.05, p.shape)
    rc = workloads.uniform_cutoffs(n, 2.5, BOUND, seed=seed)
    return (L, L, L), [dev(p[:, a]) for a in range(3)] + [dev(rc)]


def outputs(n):
    return [torch.zeros(n, **F64) for _ in range(3)] + [torch.zeros(n, dtype=torch.int32,
                                                                    device=DEV)]


def single(ctx, box, a, out, prec):
    dcm.dcm_build_cells(ctx, *a, box, EDGE, prec, rc_bound=BOUND)
    dcm.dcm_forces(ctx, dcm.make_lj(), *out[:3], prec=prec, ev_flags=dcm.DCM_EV_COUNTS,
                   nnbr=out[3])


def fresh(box, a, prec):
    out = outputs(a[0].numel())
    ctx = dcm.dcm_create()
    single(ctx, box, a, out, prec)
    assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    dcm.dcm_destroy(ctx)
    return [host(t) for t in out]


def equal(out, ref):
    for t, r in zip(out, ref):
        np.testing.assert_array_equal(host(t), r)


@pytest.mark.parametrize("prec", [dcm.DCM_FP64, dcm.DCM_FP32_MIXED])
def test_eager_build_after_a_dropped_capture(prec):
    print(f"[gpu] eager build after a dropped capture prec={prec}", flush=True)
    box, a = system(9000, 1)
    ref = fresh(box, a, prec)
    out = outputs(9000)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    poison(64 << 20)
    ctx = dcm.dcm_create(stream)
    begin(stream)
    dcm.dcm_build_cells(ctx, *a, box, EDGE, prec, rc_bound=BOUND)  # its buffers grow here
    code, g = end(stream)
    assert code == 0 and hip("hipGraphDestroy", g) == 0  # never run
    for _ in range(2):
        single(ctx, box, a, out, prec)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        equal(out, ref)
    dcm.dcm_destroy(ctx)


def test_batch_after_a_failed_capture():
    """A batch met for the first time during a capture is refused (its tables
    are uploaded and waited for); the eager call that follows is right."""
    print("[gpu] batch after a failed capture", flush=True)
    systems, refs = [], []
    for n in (3000, 9000):
        box, a = system(n, n)
        refs.append(fresh(box, a, dcm.DCM_FP64))
        out = outputs(n)
        systems.append(dict(zip(("x", "y", "z", "rc"), a), box=box, cell_edge=EDGE,
                            rc_bound=BOUND, **dict(zip(("fx", "fy", "fz", "nnbr"), out))))
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    poison(64 << 20)
    ctx = dcm.dcm_create(stream)
    begin(stream)
    with pytest.raises(dcm.DcmError):
        dcm.dcm_forces_batched(ctx, systems, dcm.make_lj(), ev_flags=dcm.DCM_EV_COUNTS)
    code, g = end(stream)
    print(f"[gpu]   capture ended with {code}", flush=True)
    if code == 0 and g:
        assert hip("hipGraphDestroy", g) == 0
    stream = torch.cuda.Stream()  # (the other one's capture may stay invalid)
    dcm.dcm_set_stream(ctx, stream)
    for graph in (False, True, True):
        for d in systems:
            d["fx"].zero_()
        torch.cuda.synchronize()
        dcm.dcm_forces_batched(ctx, systems, dcm.make_lj(), ev_flags=dcm.DCM_EV_COUNTS,
                               use_graph=graph)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        for d, ref in zip(systems, refs):
            equal([d[k] for k in ("fx", "fy", "fz", "nnbr")], ref)
    dcm.dcm_destroy(ctx)


@pytest.mark.parametrize("prec", [dcm.DCM_FP64, dcm.DCM_FP32_MIXED])
def test_replays_between_eager_builds(prec):
    print(f"[gpu] replayed builds between eager ones prec={prec}", flush=True)
    n = 9000
    box, a = system(n, 1)
    _, other = system(n, 2)
    ref, ref_other = fresh(box, a, prec), fresh(box, other, prec)
    inputs = [t.clone() for t in a]
    out, eager = outputs(n), outputs(n)
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx = dcm.dcm_create(stream)
    # more particles first: a captured build sizes its ghost buffer by an estimate
    single(ctx, box, system(13500, 3)[1], outputs(13500), prec)
    assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    single(ctx, box, other, eager, prec)
    assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    begin(stream)
    single(ctx, box, inputs, out, prec)
    code, g = end(stream)
    assert code == 0
    run = ctypes.c_void_p()
    assert hip("hipGraphInstantiate", ctypes.byref(run), g, None, None, ctypes.c_size_t(0)) == 0
    for k in range(4):
        src, want = ((a, ref), (other, ref_other))[k % 2]
        with torch.cuda.stream(stream):
            for t, s in zip(inputs, src):
                t.copy_(s)
            for t in out:
                t.zero_()
        assert hip("hipGraphLaunch", run, handle(stream)) == 0
        if k:
            single(ctx, box, other, eager, prec)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        equal(out, want)
        equal(eager, ref_other)
    assert hip("hipGraphExecDestroy", run) == 0 and hip("hipGraphDestroy", g) == 0
    dcm.dcm_destroy(ctx)


KINDS = [(dcm.DCM_PAIR_OWN, dcm.DCM_FP64), (dcm.DCM_PAIR_OWN, dcm.DCM_FP32_MIXED),
         (dcm.DCM_PAIR_MAX, dcm.DCM_FP64), (dcm.DCM_PAIR_MAX, dcm.DCM_FP32_MIXED)]


@pytest.mark.parametrize("queues", [1, 8])
def test_batch_of_every_rule_and_precision(queues):
    """Calls of every kind in turn on one context, eager, then each captured
    after a call of another kind and replayed between eager ones."""
    print(f"[gpu] batch of every kind, {queues} queues", flush=True)
    systems = []
    for n in (0, 1, 2900, 8000, 13500):
        box, a = system(n, 40 + n)
        systems.append(dict(zip(("x", "y", "z", "rc"), a), box=box, cell_edge=EDGE,
                            rc_bound=BOUND, energy=torch.zeros(1, **F64),
                            **dict(zip(("fx", "fy", "fz", "nnbr"), outputs(n)))))
    names = ("fx", "fy", "fz", "nnbr", "energy")
    flags = dcm.DCM_EV_ENERGY | dcm.DCM_EV_COUNTS

    def call(ctx, kind, graph=False):
        dcm.dcm_forces_batched(ctx, systems, dcm.make_lj(), pair_rule=kind[0], prec=kind[1],
                               ev_flags=flags, use_graph=graph)

    def check(ctx, ref):
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        for d, r in zip(systems, ref):
            equal([d[k] for k in names], r)
            for k in names:
                d[k].zero_()
        torch.cuda.synchronize()

    def fresh_batch(kind):
        ctx = dcm.dcm_create()
        dcm.dcm_set_batched_queues(ctx, queues)
        call(ctx, kind)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        dcm.dcm_destroy(ctx)
        return [[host(d[k]).copy() for k in names] for d in systems]

    refs = [fresh_batch(k) for k in KINDS]
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    ctx = dcm.dcm_create(stream)
    dcm.dcm_set_batched_queues(ctx, queues)
    for graph in (False, True):
        for kind, ref in list(zip(KINDS, refs)) * 2:
            call(ctx, kind, graph)
            check(ctx, ref)
    for k, (kind, ref) in enumerate(zip(KINDS, refs)):
        before, ref_before = KINDS[k - 1], refs[k - 1]
        call(ctx, before)
        check(ctx, ref_before)
        begin(stream)
        call(ctx, kind)
        code, g = end(stream)
        assert code == 0
        run = ctypes.c_void_p()
        assert hip("hipGraphInstantiate", ctypes.byref(run), g, None, None,
                   ctypes.c_size_t(0)) == 0
        for _ in range(3):
            assert hip("hipGraphLaunch", run, handle(stream)) == 0
            check(ctx, ref)
            call(ctx, before)
            check(ctx, ref_before)
        assert hip("hipGraphExecDestroy", run) == 0 and hip("hipGraphDestroy", g) == 0
    dcm.dcm_destroy(ctx)


# lanes per particle of the two forms: 4 and 8; 1 and 2
@pytest.mark.parametrize("n,warm,then", [
    (5000, (dcm.DCM_PAIR_OWN, dcm.DCM_FP32_MIXED), (dcm.DCM_PAIR_OWN, dcm.DCM_FP64)),
    (360000, (dcm.DCM_PAIR_MAX, dcm.DCM_FP64), (dcm.DCM_PAIR_OWN, dcm.DCM_FP64)),
])
def test_forces_of_another_form(n, warm, then):
    """Forces captured after a first call of another rule or precision."""
    print(f"[gpu] forces captured after another form n={n}", flush=True)
    rng = np.random.default_rng(n)
    m = int(np.ceil(n ** (1.0 / 3.0)))
    L = 1.1 * m
    site = rng.permutation(m ** 3)[:n]
    p = (np.stack(np.unravel_index(site, (m, m, m)), 1) + 0.5) * 1.1
    x = [dev(p[:, a]) for a in range(3)]
    rc = dev(workloads.uniform_cutoffs(n, 2.5, 4.0, seed=1))
    out = outputs(n)

    def forces(ctx, form, o):
        dcm.dcm_forces(ctx, dcm.make_lj(), *o[:3], pair_rule=form[0], prec=form[1],
                       ev_flags=dcm.DCM_EV_COUNTS, nnbr=o[3])

    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    refs = []
    for form in (warm, then):
        ctx = dcm.dcm_create(stream)
        dcm.dcm_build_cells(ctx, *x, rc, (L, L, L), EDGE, dcm.DCM_FP32_MIXED, rc_bound=4.0)
        forces(ctx, form, out)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        refs.append([host(t).copy() for t in out])
        dcm.dcm_destroy(ctx)
    ctx = dcm.dcm_create(stream)
    dcm.dcm_build_cells(ctx, *x, rc, (L, L, L), EDGE, dcm.DCM_FP32_MIXED, rc_bound=4.0)
    forces(ctx, warm, out)
    assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
    equal(out, refs[0])
    begin(stream)
    forces(ctx, then, out)
    code, g = end(stream)
    assert code == 0
    run = ctypes.c_void_p()
    assert hip("hipGraphInstantiate", ctypes.byref(run), g, None, None, ctypes.c_size_t(0)) == 0
    for _ in range(3):
        assert hip("hipGraphLaunch", run, handle(stream)) == 0
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        equal(out, refs[1])
        forces(ctx, warm, out)
        assert dcm.dcm_sync_status(ctx) == dcm.DCM_OK
        equal(out, refs[0])
    assert hip("hipGraphExecDestroy", run) == 0 and hip("hipGraphDestroy", g) == 0
    dcm.dcm_destroy(ctx)
