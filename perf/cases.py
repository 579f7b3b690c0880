"""Performance cases of the dynamic cutoff method library: the work its users
have it do, through the entry points of ``paper_1701_05242_amd``.

Five kinds of case:

* ``step``: a molecular dynamics run that takes ``nsteps`` steps with dcm_step
  and then has the state in hand (the main path; small systems are bound by
  latency and launches, large ones by the pair kernel and the grid stages);
* ``forces``: linked cells and forces of one snapshot (dcm_build_cells,
  dcm_forces), as a program with an integrator of its own calls them;
* ``interface``: detection, distance field and cutoffs of one snapshot
  (dcm_detect_interface[_opts], dcm_sweep_distance, dcm_assign_cutoffs);
* ``list``: a step on a stored Verlet list (dcm_update_list, dcm_forces_list);
* ``batch``: cells and forces of many independent systems at once
  (dcm_forces_batched).

Systems are liquid/vapour slabs, droplets and cylinders at reduced densities
0.8 and 0.02: a face-centred cubic liquid displaced by about the thermal
displacement near melting, a vapour without overlaps, Maxwell-Boltzmann
velocities at T* = 0.7.  The particle count follows from the geometry alone.

FP32-mixed results carry single-precision rounding; their programs keep what
comes out of a pass as a single-precision frame, as trajectory files hold it.
"""
import math

import numpy as np
import torch

import paper_1701_05242_amd as dcm

RHO_L, RHO_V, T_STAR = 0.8, 0.02, 0.7
RAMP = 5.0
DT = 0.005
F64 = torch.float64


def listed():
    slab = dict(geom="slab", rc_min=2.5)
    return [
        # the smallest run: a 3,000-particle slab in double precision, interface
        # found anew every step; every launch and every wait counts
        dict(slab, name="step_slab_3k_fp64", kind="step", lx=13.4, ly=13.4, lz=60.0, liquid=20.0,
             rc_max=6.0, prec="fp64", nsteps=20, redetect=1, energy=False),
        # the size of the accuracy experiment (about 20,000 particles, wide cutoffs)
        dict(slab, name="step_slab_20k_mixed", kind="step", lx=26.8, ly=26.8, lz=90.0,
             liquid=33.0, rc_min=3.0, rc_max=8.0, prec="mixed", nsteps=10, redetect=10,
             energy=False),
        # a constant-energy run that records its energies every step
        dict(slab, name="step_slab_99k_fp64_nve", kind="step", lx=54.0, ly=54.0, lz=120.0,
             liquid=40.0, rc_max=6.0, prec="fp64", nsteps=10, redetect=10, energy=True),
        # a droplet: curved interface, a grid large against its particles
        dict(name="step_droplet_122k_mixed", kind="step", geom="droplet", lx=120.0, ly=120.0,
             lz=120.0, liquid=30.0, rc_min=2.5, rc_max=8.0, prec="mixed", nsteps=5, redetect=1,
             energy=False),
        # a cylinder in double precision
        dict(name="step_cylinder_341k_fp64", kind="step", geom="cylinder", lx=200.0, ly=100.0,
             lz=100.0, liquid=25.0, rc_min=2.5, rc_max=8.0, prec="fp64", nsteps=5, redetect=1,
             energy=False),
        # a production-size slab in double precision, interface found every tenth step
        dict(slab, name="step_slab_1200k_fp64", kind="step", lx=120.0, ly=120.0, lz=250.0,
             liquid=100.0, rc_min=3.0, rc_max=8.0, prec="fp64", nsteps=10, redetect=10,
             energy=False),
        # the headline run: 2.6 million particles, mixed precision, interface every step
        dict(slab, name="step_slab_2600k_mixed", kind="step", lx=160.0, ly=160.0, lz=400.0,
             liquid=120.0, rc_max=8.0, prec="mixed", nsteps=4, redetect=1, energy=False),
        # forces, energy, virial and neighbour counts under the symmetric rule
        dict(slab, name="forces_slab_99k_max_fp64", kind="forces", lx=54.0, ly=54.0, lz=120.0,
             liquid=40.0, rc_max=6.0, prec="fp64", rule="max", observables=True),
        # interface analysis of one large snapshot
        dict(slab, name="interface_slab_2600k", kind="interface", lx=160.0, ly=160.0, lz=400.0,
             liquid=120.0, rc_max=8.0, nu=-1.0, min_volume=0),
        # one step on a stored list with a skin
        dict(slab, name="list_slab_99k_fp64", kind="list", lx=54.0, ly=54.0, lz=120.0,
             liquid=40.0, rc_max=6.0, prec="fp64", skin=0.3),
        # 64 independent slabs of 2,000 to 200,000 particles, one recorded graph
        dict(name="batch_64_mixed", kind="batch", count=64, n_min=2000, n_max=200000,
             prec="mixed", graph=True, observables=False),
        # a few small systems with every observable, called eagerly
        dict(name="batch_12_fp64", kind="batch", count=12, n_min=2000, n_max=20000, prec="fp64",
             graph=False, observables=True),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _drawn_box(rng, n, rc_max):
    """A box and a liquid of one of the three geometries for about n particles."""
    low = 2.0 * rc_max + 0.5
    geom = rng.choice(("slab", "slab", "droplet", "cylinder")) if n >= 20000 else "slab"
    if geom == "slab":
        share, aspect = rng.uniform(0.3, 0.45), rng.uniform(1.2, 4.5)
        vol = n / (share * RHO_L + (1.0 - share) * RHO_V)
        lx = max(low, (vol / aspect) ** (1.0 / 3.0))
        ly = max(low, lx * rng.uniform(0.9, 1.1))
        lz = max(low, vol / (lx * ly))
        liquid = share * lz
    elif geom == "droplet":
        part = rng.uniform(0.22, 0.3)          # radius over the edge
        share = 4.0 / 3.0 * math.pi * part ** 3
        lx = max(low, (n / (share * RHO_L + (1.0 - share) * RHO_V)) ** (1.0 / 3.0))
        ly = lz = lx
        liquid = part * lx
    else:
        part, aspect = rng.uniform(0.22, 0.3), rng.uniform(0.7, 2.5)
        share = math.pi * part ** 2
        ly = max(low, (n / (share * RHO_L + (1.0 - share) * RHO_V) / aspect) ** (1.0 / 3.0))
        lx, lz = max(low, aspect * ly), ly
        liquid = part * ly
    return dict(geom=geom, lx=round(lx, 2), ly=round(ly, 2), lz=round(lz, 2),
                liquid=round(liquid, 2))


def draw(rng):
    kind = rng.choice(("step",) * 6 + ("forces", "interface", "list", "batch"))
    prec = rng.choice(("fp64", "mixed"))
    rc_min, rc_max = round(rng.uniform(2.5, 3.2), 2), round(rng.uniform(4.0, 8.0), 2)
    base = dict(kind=kind, rc_min=rc_min, rc_max=rc_max)
    if kind == "step":
        n = _log(rng, 2000, 1.2e6 if prec == "fp64" else 2.5e6)
        return dict(base, **_drawn_box(rng, n, rc_max), prec=prec,
                    nsteps=max(2, min(20, int(4e6 / n))), redetect=rng.choice((1, 1, 5, 10)),
                    energy=rng.random() < 0.3)
    if kind == "forces":
        n = _log(rng, 2000, 2.5e6)
        rule = "max" if n < 1.2e5 and rng.random() < 0.4 else "own"
        return dict(base, **_drawn_box(rng, n, rc_max), prec=prec, rule=rule,
                    observables=rng.random() < 0.5)
    if kind == "interface":
        opts = rng.random() < 0.4
        return dict(base, **_drawn_box(rng, _log(rng, 2000, 2.5e6), rc_max),
                    nu=round(rng.uniform(0.5, 8.0), 2) if opts else -1.0,
                    min_volume=rng.choice((0, 40)) if opts else 0)
    if kind == "list":
        return dict(base, **_drawn_box(rng, _log(rng, 2000, 3e5), rc_max), prec=prec,
                    skin=round(rng.uniform(0.1, 0.4), 2))
    n_max = int(_log(rng, 5000, 2e5))
    return dict(kind="batch", count=rng.randint(3, max(3, min(64, int(1.5e6 / n_max)))),
                n_min=2000, n_max=n_max, prec=prec, graph=rng.random() < 0.5,
                observables=rng.random() < 0.5)


# ------------------------------------------------------------------ systems

def _box(case):
    return (case["lx"], case["ly"], case["lz"])


def _batch_systems(case):
    """The systems of a batch: log-spaced sizes, cutoffs of 4 to 8 in turn."""
    out = []
    for b in range(case["count"]):
        t = (b + 0.5) / case["count"]
        n = case["n_min"] * (case["n_max"] / case["n_min"]) ** t
        rc_max = 4.0 + 4.0 * ((b * 0.6180339887) % 1.0)
        low = 2.0 * rc_max + 0.5
        rho = RHO_L / 3.0 + 2.0 * RHO_V / 3.0
        lxy = max(low, (n / (rho * 60.0 / 13.4)) ** (1.0 / 3.0))
        lz = max(low, n / (rho * lxy * lxy))
        out.append(dict(geom="slab", lx=lxy, ly=lxy, lz=lz, liquid=lz / 3.0, rc_min=2.5,
                        rc_max=rc_max))
    return out


def _lattice(counts, steps, basis, dev):
    i = torch.cartesian_prod(*(torch.arange(c, dtype=F64, device=dev) for c in counts))
    p = (i.reshape(-1, 1, 3) + basis).reshape(-1, 3)
    return p * torch.tensor(steps, dtype=F64, device=dev)


def _inside(case, p, grown=0.0):
    """Which points lie in the liquid grown by `grown`."""
    c = torch.tensor(_box(case), dtype=F64, device=p.device) / 2.0
    if case["geom"] == "slab":
        return (p[:, 2] - c[2]).abs() < case["liquid"] / 2.0 + grown
    axes = (0, 1, 2) if case["geom"] == "droplet" else (1, 2)
    r2 = sum((p[:, a] - c[a]) ** 2 for a in axes)
    return r2 < (case["liquid"] + grown) ** 2


def _particles(case, gen, dev):
    """Positions [3, n] inside the box."""
    box = _box(case)
    a0 = (4.0 / RHO_L) ** (1.0 / 3.0)
    fcc = torch.tensor([[0.25, 0.25, 0.25], [0.75, 0.75, 0.25], [0.75, 0.25, 0.75],
                        [0.25, 0.75, 0.75]], dtype=F64, device=dev)
    ext = list(box)
    if case["geom"] == "slab":
        ext[2] = case["liquid"]
    k = [max(1, round(e / a0)) for e in ext]
    liq = _lattice(k, [e / m for e, m in zip(ext, k)], fcc, dev)
    if case["geom"] == "slab":
        liq[:, 2] += (box[2] - case["liquid"]) / 2.0
    liq = liq[_inside(case, liq)]
    liq += (torch.rand(liq.shape, generator=gen, dtype=F64, device=dev) - 0.5) * 0.2
    # vapour: some sites of a wide simple cubic lattice outside the liquid
    m = [max(1, int(b / 1.3)) for b in box]
    site = torch.full((1, 3), 0.5, dtype=F64, device=dev)
    vap = _lattice(m, [b / q for b, q in zip(box, m)], site, dev)
    vap = vap[~_inside(case, vap, 1.1)]
    vol = box[0] * box[1] * box[2] - liq.shape[0] / RHO_L
    take = min(vap.shape[0], int(round(RHO_V * vol)))
    vap = vap[torch.randperm(vap.shape[0], generator=gen, device=dev)[:take]]
    vap += (torch.rand(vap.shape, generator=gen, dtype=F64, device=dev) - 0.5) * 0.3
    p = torch.cat([liq, vap])
    L = torch.tensor(box, dtype=F64, device=dev)
    p = p - L * torch.floor(p / L)
    return torch.where(p >= L, torch.zeros_like(p), p).T.contiguous()


def _velocities(n, gen, dev):
    v = torch.randn((3, n), generator=gen, dtype=F64, device=dev) * math.sqrt(T_STAR)
    return v - v.mean(dim=1, keepdim=True)


def _generator(case, seed):
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    return gen, dev


# ------------------------------------------------------------------ the passes

class _Handle:
    """A library context that goes with the state that holds it."""

    def __init__(self):
        self.ctx = dcm.dcm_create()

    def __del__(self):
        if getattr(self, "ctx", None) is not None:
            dcm.dcm_destroy(self.ctx)
            self.ctx = None


_PREC = {"fp64": dcm.DCM_FP64, "mixed": dcm.DCM_FP32_MIXED}
_RULE = {"own": dcm.DCM_PAIR_OWN, "max": dcm.DCM_PAIR_MAX}


def _cutoffs_from_interface(case, ctx, p, dev):
    """Detection, distance field and cutoffs into new arrays."""
    box = _box(case)
    grid = dcm.make_grid(box, 1.0)
    rule = dcm.make_rule(case["rc_min"], case["rc_max"], RAMP)
    nv = dcm.grid_voxels(grid)
    seg = torch.empty(nv, dtype=torch.uint8, device=dev)
    iface = torch.empty(nv, dtype=torch.uint8, device=dev)
    dist = torch.empty(nv, dtype=F64, device=dev)
    delta, rc = (torch.empty(p.shape[1], dtype=F64, device=dev) for _ in range(2))
    dcm.dcm_detect_interface(ctx, *p, box, grid, seg, iface)
    dcm.dcm_sweep_distance(ctx, seg, iface, grid, dcm.dcm_rc_grid(rule, grid), 64, dist)
    dcm.dcm_assign_cutoffs(ctx, *p, box, grid, dist, rule, rc, delta)
    return rc


def prepare(case, seed):
    gen, dev = _generator(case, seed)
    kind = case["kind"]
    st = dict(case=case, handle=_Handle(), lj=dcm.make_lj())
    ctx = st["handle"].ctx
    if kind == "batch":
        systems, cases = [], _batch_systems(case)
        pos = [_particles(c, gen, dev) for c in cases]
        total = sum(p.shape[1] for p in pos)
        nsys = len(pos)
        st["F"] = torch.zeros((3, total), dtype=F64, device=dev)
        st["E"] = torch.zeros(nsys, dtype=F64, device=dev)
        st["W"] = torch.zeros((nsys, 6), dtype=F64, device=dev)
        st["nnbr"] = torch.zeros(total, dtype=torch.int32, device=dev)
        st["npairs"] = torch.zeros(nsys, dtype=torch.int64, device=dev)
        npairs = st["npairs"].view(torch.uint64)
        st["keep"], at = [pos], 0
        for b, (c, p) in enumerate(zip(cases, pos)):
            n = p.shape[1]
            rc = _cutoffs_from_interface(c, ctx, p, dev)
            st["keep"].append(rc)
            d = dict(x=p[0], y=p[1], z=p[2], rc=rc, fx=st["F"][0, at:at + n],
                     fy=st["F"][1, at:at + n], fz=st["F"][2, at:at + n], box=_box(c),
                     rc_bound=c["rc_max"], energy=st["E"][b:b + 1])
            if case["observables"]:
                d.update(virial=st["W"][b], nnbr=st["nnbr"][at:at + n], npairs=npairs[b:b + 1])
            systems.append(d)
            at += n
        st["systems"] = dcm.make_systems(systems)
        return st
    p = _particles(case, gen, dev)
    n, box = p.shape[1], _box(case)
    f = torch.zeros((3, n), dtype=F64, device=dev)
    if kind == "step":
        # x y z, vx vy vz, fx fy fz of a run, with the forces at its start
        st["S"] = torch.cat([p, _velocities(n, gen, dev), f])
        st["grid"] = dcm.make_grid(box, 1.0)
        st["rule"] = dcm.make_rule(case["rc_min"], case["rc_max"], RAMP)
        st["rc_grid"] = dcm.dcm_rc_grid(st["rule"], st["grid"])
        st["series"] = (torch.zeros(2 * case["nsteps"], dtype=F64, device=dev)
                        if case["energy"] else None)
        st["done"] = 0
        dcm.dcm_step(ctx, *st["S"], box, st["lj"], st["rule"], st["grid"], st["rc_grid"], DT, 0,
                     prec=_PREC[case["prec"]])
        return st
    st["p"] = p
    if kind == "interface":
        st["grid"] = dcm.make_grid(box, 1.0)
        st["rule"] = dcm.make_rule(case["rc_min"], case["rc_max"], RAMP)
        st["rc_grid"] = dcm.dcm_rc_grid(st["rule"], st["grid"])
        nv = dcm.grid_voxels(st["grid"])
        st["seg"] = torch.empty(nv, dtype=torch.uint8, device=dev)
        st["iface"] = torch.empty(nv, dtype=torch.uint8, device=dev)
        st["dist"] = torch.empty(nv, dtype=F64, device=dev)
        st["delta"], st["rc"] = (torch.empty(n, dtype=F64, device=dev) for _ in range(2))
        return st
    st["rc"] = _cutoffs_from_interface(case, ctx, p, dev)
    st["F"] = f
    if kind == "forces":
        st["E"] = torch.zeros(1, dtype=F64, device=dev)
        st["W"] = torch.zeros(6, dtype=F64, device=dev)
        st["nnbr"] = torch.zeros(n, dtype=torch.int32, device=dev)
        st["npairs"] = torch.zeros(1, dtype=torch.int64, device=dev)
        return st
    # list: built at p; the step's positions lie a little off
    prec = _PREC[case["prec"]]
    dcm.dcm_build_cells(ctx, *p, st["rc"], box, 1.25, prec, rc_bound=case["rc_max"])
    dcm.dcm_build_list(ctx, case["skin"])
    L = torch.tensor(box, dtype=F64, device=dev).reshape(3, 1)
    q = p + (torch.rand(p.shape, generator=gen, dtype=F64, device=dev) - 0.5) * case["skin"] * 0.5
    q = q - L * torch.floor(q / L)
    st["q"] = torch.where(q >= L, torch.zeros_like(q), q)
    return st


def run(st):
    case, ctx, kind = st["case"], st["handle"].ctx, st["case"]["kind"]
    mixed = case.get("prec") == "mixed"
    if kind == "step":
        dcm.dcm_step(ctx, *st["S"], _box(case), st["lj"], st["rule"], st["grid"], st["rc_grid"],
                     DT, case["nsteps"], prec=_PREC[case["prec"]],
                     redetect_every=case["redetect"], step0=st["done"],
                     energy_series=st["series"])
        st["done"] += case["nsteps"]
        S = st["S"].float() if mixed else st["S"]
        out = dict(x=S[:3], v=S[3:6], F=S[6:])
        if case["energy"]:
            out["series"] = st["series"].float() if mixed else st["series"]
        return out
    if kind == "interface":
        args = (ctx, *st["p"], _box(case), st["grid"], st["seg"], st["iface"])
        if case["nu"] >= 0.0 or case["min_volume"]:
            dcm.dcm_detect_interface_opts(*args, nu=case["nu"], min_volume=case["min_volume"])
        else:
            dcm.dcm_detect_interface(*args)
        dcm.dcm_sweep_distance(ctx, st["seg"], st["iface"], st["grid"], st["rc_grid"], 64,
                               st["dist"])
        dcm.dcm_assign_cutoffs(ctx, *st["p"], _box(case), st["grid"], st["dist"], st["rule"],
                               st["rc"], st["delta"])
        return {k: st[k] for k in ("seg", "iface", "dist", "delta", "rc")}
    if kind == "list":
        dcm.dcm_update_list(ctx, *st["q"], st["rc"])
        dcm.dcm_forces_list(ctx, st["lj"], *st["F"], prec=_PREC[case["prec"]])
        return dict(F=st["F"].float() if mixed else st["F"])
    flags = dcm.DCM_EV_ENERGY
    if case["observables"]:
        flags |= dcm.DCM_EV_VIRIAL | dcm.DCM_EV_COUNTS
    if kind == "forces":
        dcm.dcm_build_cells(ctx, *st["p"], st["rc"], _box(case), 0.0, _PREC[case["prec"]],
                            rc_bound=case["rc_max"])
        more = (dict(virial=st["W"], nnbr=st["nnbr"], npairs=st["npairs"].view(torch.uint64))
                if case["observables"] else {})
        dcm.dcm_forces(ctx, st["lj"], *st["F"], pair_rule=_RULE[case["rule"]],
                       prec=_PREC[case["prec"]], ev_flags=flags, energy=st["E"], **more)
    else:
        dcm.dcm_forces_batched(ctx, st["systems"], st["lj"], prec=_PREC[case["prec"]],
                               ev_flags=flags, use_graph=case["graph"])
    keys = ("F", "E") + (("W", "nnbr", "npairs") if case["observables"] else ())
    return {k: st[k].float() if mixed and st[k].is_floating_point() else st[k] for k in keys}


# ------------------------------------------------------------------ the least work

def _estimate(case):
    """Particles, interacting ordered pairs (own rule) and voxels, from the geometry."""
    lx, ly, lz = _box(case)
    vol, r = lx * ly * lz, case["liquid"]
    if case["geom"] == "slab":
        v_l, area, deep = lx * ly * r, 2.0 * lx * ly, r / 2.0
    elif case["geom"] == "droplet":
        v_l, area, deep = 4.0 / 3.0 * math.pi * r ** 3, 4.0 * math.pi * r * r, r / 3.0
    else:
        v_l, area, deep = math.pi * r * r * lx, 2.0 * math.pi * r * lx, r / 2.0
    n = RHO_L * v_l + RHO_V * (vol - v_l)

    def sphere(rc, s):  # neighbours of a particle at depth s below a flat interface
        full, cap = 4.0 / 3.0 * math.pi * rc ** 3, 0.0
        if s < rc:
            h = rc - s
            cap = math.pi * h * h * (3.0 * rc - h) / 3.0
        return RHO_L * (full - cap) + RHO_V * cap

    slices, top, pairs = 40, min(RAMP, deep), 0.0
    for k in range(slices):
        s = (k + 0.5) * top / slices
        rc = case["rc_max"] - (case["rc_max"] - case["rc_min"]) * min(s / RAMP, 1.0)
        pairs += RHO_L * area * top / slices * sphere(rc, s)
    pairs += RHO_L * max(0.0, v_l - area * top) * sphere(case["rc_min"], 1e9)
    pairs += RHO_V * (vol - v_l) * RHO_V * 4.0 / 3.0 * math.pi * case["rc_max"] ** 3
    return n, pairs, vol


def work(case):
    """24 operations for each interacting pair with its energy.  Bytes: a step
    reads and writes positions, velocities and forces (72 bytes each way); a
    force pass reads positions and cutoffs and writes forces; an interface
    pass reads positions, writes two bytes and a distance for each voxel, and
    a distance and a cutoff for each particle."""
    if case["kind"] == "batch":
        e = [_estimate(c) for c in _batch_systems(case)]
        return dict(bytes=56.0 * sum(v[0] for v in e), flops=24.0 * sum(v[1] for v in e))
    n, pairs, voxels = _estimate(case)
    if case["kind"] == "step":
        return dict(bytes=144.0 * n * case["nsteps"], flops=24.0 * pairs * case["nsteps"])
    if case["kind"] == "interface":
        return dict(bytes=40.0 * n + 10.0 * voxels, flops=0.0)
    if case.get("rule") == "max":
        pairs *= 1.15  # pairs found from the other end only
    return dict(bytes=56.0 * n, flops=24.0 * pairs)


# ------------------------------------------------- the method in plain 64 bits

def _phases(case, p):
    """Phase map and grid of the two-phase split, regularised."""
    box = _box(case)
    nv = [max(1, int(math.floor(b + 0.5))) for b in box]
    idx = [(p[a] * (nv[a] / box[a])).floor().long().clamp(0, nv[a] - 1) for a in range(3)]
    flat = (idx[2] * nv[1] + idx[1]) * nv[0] + idx[0]
    g = torch.bincount(flat, minlength=nv[0] * nv[1] * nv[2]).reshape(nv[2], nv[1], nv[0])

    def window(t):
        for d in range(3):
            t = t + torch.roll(t, 1, d) + torch.roll(t, -1, d)
        return t

    g = window(g)
    h = torch.bincount(g.reshape(-1)).double().cpu().numpy()
    t = np.arange(len(h))
    n1, s1 = np.cumsum(h[::-1])[::-1], np.cumsum((h * t)[::-1])[::-1]
    n0, s0 = h.sum() - n1, (h * t).sum() - s1
    ok = (n0 > 0) & (n1 > 0)
    score = np.full(len(h), -1.0)
    score[ok] = s0[ok] ** 2 / n0[ok] + s1[ok] ** 2 / n1[ok]
    thr = int(np.argmax(score))
    c0, c1 = s0[thr] / n0[thr], s1[thr] / n1[thr]
    seg = g >= thr
    before = None
    nu = case.get("nu", -1.0)
    for _ in range(16):
        around = window(seg.int())
        if nu >= 0.0:
            d = ((g - c1) ** 2 - (g - c0) ** 2) + nu * (26 - 2 * (around - seg.int()))
            new = torch.where(d == 0, seg, d < 0)
        else:
            new = around >= 14
        stop = torch.equal(new, seg) or (before is not None and torch.equal(new, before))
        before, seg = seg, new
        if stop:
            break
    if case.get("min_volume", 0):
        # components of both phases: the smallest voxel number spreads over faces
        lab = torch.arange(seg.numel(), device=seg.device).reshape(seg.shape)
        while True:
            new = lab
            for d in range(3):
                for s in (1, -1):
                    o = torch.roll(new, s, d)
                    new = torch.where(torch.roll(seg, s, d) == seg, torch.minimum(new, o), new)
            new = new.reshape(-1)[new.reshape(-1)].reshape(seg.shape)
            if torch.equal(new, lab):
                break
            lab = new
        size = torch.bincount(lab.reshape(-1), minlength=seg.numel())[lab]
        seg = torch.where(size < case["min_volume"], ~seg, seg)
    return seg, nv


def _distances(case, seg, nv):
    """|grad d| = 1 upwind from the low-density phase and the interface, up to rc_grid."""
    box = _box(case)
    h = [box[a] / nv[a] for a in range(3)]
    rc_grid = RAMP + 3.0 * max(h)
    face = seg.clone()
    for d in range(3):
        face &= torch.roll(seg, 1, d) & torch.roll(seg, -1, d)
    D = torch.where(face, math.inf, 0.0).to(F64)
    hs = torch.tensor(h, dtype=F64, device=D.device)
    inf = torch.tensor(math.inf, dtype=F64, device=D.device)
    while True:
        at = torch.nonzero((D > 0.0).reshape(-1)).reshape(-1)
        near = [torch.minimum(torch.roll(D, 1, 2 - a), torch.roll(D, -1, 2 - a)).reshape(-1)[at]
                for a in range(3)]
        a, order = torch.sort(torch.stack(near), dim=0, stable=True)
        live = torch.isfinite(a[0])
        at, a, hk = at[live], a[:, live], hs[order[:, live]]
        w = 1.0 / hk ** 2
        d1 = a[0] + hk[0]
        b1 = torch.where(torch.isfinite(a[1]), a[1] - a[0], 0.0)
        b2 = torch.where(torch.isfinite(a[2]), a[2] - a[0], 0.0)

        def root(A, B, C):
            return a[0] + (B + torch.sqrt((B * B - A * C).clamp(min=0.0))) / A

        d2 = root(w[0] + w[1], w[1] * b1, w[1] * b1 ** 2 - 1.0)
        d3 = root(w[0] + w[1] + w[2], w[1] * b1 + w[2] * b2,
                  w[1] * b1 ** 2 + w[2] * b2 ** 2 - 1.0)
        g = torch.where(d1 <= a[1], d1, torch.where(d2 <= a[2], d2, d3))
        old = D.reshape(-1)[at]
        new = torch.where((g < old) & (g <= rc_grid), g, old)
        if torch.equal(new, old):
            return torch.minimum(D, inf.clamp(max=rc_grid))
        D.reshape(-1)[at] = new


def _cutoffs(case, p, D):
    box, nv = _box(case), D.shape[::-1]
    lo, hi, t = [], [], []
    for a in range(3):
        u = p[a] * (nv[a] / box[a]) - 0.5
        f = torch.floor(u)
        t.append(u - f)
        lo.append(f.long() % nv[a])
        hi.append((f.long() + 1) % nv[a])
    d = 0.0
    for k, wz in ((lo[2], 1 - t[2]), (hi[2], t[2])):
        for j, wy in ((lo[1], 1 - t[1]), (hi[1], t[1])):
            for i, wx in ((lo[0], 1 - t[0]), (hi[0], t[0])):
                d = d + D[k, j, i] * wx * wy * wz
    rc = case["rc_max"] - (case["rc_max"] - case["rc_min"]) * (d / RAMP).clamp(max=1.0)
    return d, rc


def _forces(case, p, rc, rule="own"):
    """F [3, n], energy, virial [6] and pair counts over every pair of the rule."""
    box, dev, n, edge = _box(case), p.device, p.shape[1], 1.25
    reach = float(rc.max())
    q, src = p, torch.arange(n, device=dev)
    for a in range(3):  # periodic images within reach of the box
        up, dn = q[a] < reach, q[a] >= box[a] - reach
        shift = torch.zeros((3, 1), dtype=F64, device=dev)
        shift[a] = box[a]
        q, src = (torch.cat([q, q[:, up] + shift, q[:, dn] - shift], 1),
                  torch.cat([src, src[up], src[dn]]))
    pad = int(math.ceil(reach / edge)) + 1
    nc = [int(math.floor(b / edge)) + 1 + 2 * pad for b in box]
    cell = [(q[a] / edge).floor().long() + pad for a in range(3)]
    flat = (cell[2] * nc[1] + cell[1]) * nc[0] + cell[0]
    flat, order = torch.sort(flat)
    q, src = q[:, order].contiguous(), src[order]
    start = torch.searchsorted(flat, torch.arange(nc[0] * nc[1] * nc[2] + 1, device=dev))
    home = [(p[a] / edge).floor().long() + pad for a in range(3)]
    F = torch.zeros((3, n), dtype=F64, device=dev)
    E = torch.zeros((), dtype=F64, device=dev)
    W = torch.zeros(6, dtype=F64, device=dev)
    nn = torch.zeros(n, dtype=torch.int64, device=dev)
    search = torch.full_like(rc, reach) if rule == "max" else rc
    ring = torch.ceil(search / edge).long()
    for k in torch.unique(ring).tolist():
        group = torch.nonzero(ring == k).reshape(-1)
        for dz in range(-k, k + 1):
            for dy in range(-k, k + 1):
                if max(abs(dz) - 1, 0) ** 2 + max(abs(dy) - 1, 0) ** 2 > k * k:
                    continue
                row = ((home[2][group] + dz) * nc[1] + home[1][group] + dy) * nc[0] + home[0][group]
                a, b = start[row - k], start[row + k + 1]
                for part in torch.split(torch.arange(group.numel(), device=dev), 1 << 18):
                    cnt = b[part] - a[part]
                    i = torch.repeat_interleave(group[part], cnt)
                    first = torch.repeat_interleave(a[part] - (torch.cumsum(cnt, 0) - cnt), cnt)
                    j = first + torch.arange(i.numel(), device=dev)
                    d = p[:, i] - q[:, j]
                    r2 = (d * d).sum(0)
                    if rule == "max":
                        hit = r2 <= torch.maximum(rc[i], rc[src[j]]) ** 2
                    else:
                        hit = r2 < rc[i] ** 2
                    hit &= ~((src[j] == i) & (r2 == 0.0))
                    i, d, r2 = i[hit], d[:, hit], r2[hit]
                    s6 = 1.0 / r2 ** 3
                    f = 24.0 * s6 * (2.0 * s6 - 1.0) / r2 * d
                    for c in range(3):
                        F[c].index_add_(0, i, f[c])
                    nn.index_add_(0, i, torch.ones_like(i))
                    E += (2.0 * s6 * (s6 - 1.0)).sum()
                    for c, (u, v) in enumerate(((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))):
                        W[c] += 0.5 * (d[u] * f[v]).sum()
    return F, E, W, nn


def exact(case, seed):
    gen, dev = _generator(case, seed)
    kind = case["kind"]
    if kind == "batch":
        cases = _batch_systems(case)
        pos = [_particles(c, gen, dev) for c in cases]
        got = []
        for c, p in zip(cases, pos):
            D = _distances(c, *_phases(c, p))
            got.append(_forces(c, p, _cutoffs(c, p, D)[1]))
        out = dict(F=torch.cat([g[0] for g in got], 1), E=torch.stack([g[1] for g in got]))
        if case["observables"]:
            out.update(W=torch.stack([g[2] for g in got]), nnbr=None, npairs=None)
        return out
    p = _particles(case, gen, dev)
    if kind == "interface":
        seg, nv = _phases(case, p)
        D = _distances(case, seg, nv)
        delta, rc = _cutoffs(case, p, D)
        return dict(seg=None, iface=None, dist=D.reshape(-1), delta=delta, rc=rc)
    D = _distances(case, *_phases(case, p))
    rc = _cutoffs(case, p, D)[1]
    if kind == "list":
        L = torch.tensor(_box(case), dtype=F64, device=dev).reshape(3, 1)
        q = p + (torch.rand(p.shape, generator=gen, dtype=F64, device=dev) - 0.5) * case["skin"] * 0.5
        q = q - L * torch.floor(q / L)
        return dict(F=_forces(case, torch.where(q >= L, torch.zeros_like(q), q), rc)[0])
    if kind == "forces":
        F, E, W, nn = _forces(case, p, rc, case["rule"])
        out = dict(F=F, E=E.reshape(1))
        if case["observables"]:
            out.update(W=W, nnbr=None, npairs=None)
        return out
    v = _velocities(p.shape[1], gen, dev)
    L = torch.tensor(_box(case), dtype=F64, device=dev).reshape(3, 1)
    F = _forces(case, p, rc)[0]
    series = []
    for s in range(case["nsteps"]):
        v = v + 0.5 * DT * F
        p = p + DT * v
        p = p - L * torch.floor(p / L)
        p = torch.where(p >= L, torch.zeros_like(p), p)
        if (s + 1) % case["redetect"] == 0:
            D = _distances(case, *_phases(case, p))
        F, E, _, _ = _forces(case, p, _cutoffs(case, p, D)[1])
        v = v + 0.5 * DT * F
        series += [E, 0.5 * (v * v).sum()]
    out = dict(x=p, v=v, F=F)
    if case["energy"]:
        out["series"] = torch.stack(series)
    return out
