"""Work that programs have this framework do, as cases that can be timed.

    listed()             the cases, dicts of plain values
    draw(rng)            one more case of the same ranges
    prepare(case, seed)  what a program holds before the call (simulation, trajectory, shells)
    run(state)           one pass through the public entry points, and its outputs
    work(case)           bytes and operations a pass cannot do without
    exact(case, seed)    what run returns, in plain torch FP64 (None where it takes too long)

Kinds of work:

    step        advance a simulation by `steps` fluid steps and read its state (fields, bodies):
                one recording interval of a run
    resistance  the Stokes-flow measurement: `samples` times 10 steps and the drag
    adjoint     the reverse pass over a window of steps (gradients by friction and bead offsets)
    analysis    every series and mean squared displacement of a recorded trajectory
    construct   relax the bead shells of raspberries

The simulations are the ones of the paper and of paper_1604_01829_amd.workloads -- the same
boxes, shells, frictions and noise -- with seeds of their own, warmed up so that the fluid moves.
"""
import math

import numpy as np
import torch

from paper_1604_01829_amd import analysis as A
from paper_1604_01829_amd import construction as C
from paper_1604_01829_amd import lbrb
from paper_1604_01829_amd import workloads as W

KT = 4e-5                # the workloads' thermal energy
WARM = 100               # steps of a simulation before the first pass
DEVICE = "cuda:0"


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # smallest: one free sphere in a 32^3 box, FP64, driven and deterministic; launches and
        # latency count
        dict(name="sphere32_f64", kind="step", wall="none", nx=32, ny=32, nz=32, bodies=1,
             radius=3.0, precision="f64", thermal=False, steps=100),
        # the paper's Stokes-flow set-up: 50^3 channel between moving walls, a fixed sphere, the
        # drag read every 10 steps (short calls, eager launches, results on the host)
        dict(name="stokes50_f64", kind="resistance", nx=50, radius=5.25, samples=10),
        # ordinary: spheres in a long pore, FP32, thermal; the populations fit in the cache
        dict(name="pore128_f32", kind="step", wall="pore", nx=128, ny=128, nz=256, bodies=32,
             radius=4.0, precision="f32", thermal=True, steps=100),
        # the same pore in the paper's integration scheme: two MD steps per fluid step, inner
        # excluded-volume layers and pore beads
        dict(name="confined128_f32", kind="step", wall="confined", nx=128, ny=128, nz=256,
             bodies=32, radius=4.0, precision="f32", thermal=True, steps=100),
        # largest box: ellipsoids in 256^3, FP32, thermal; far beyond the caches
        dict(name="box256_f32", kind="step", wall="none", nx=256, ny=256, nz=256, bodies=16,
             radius=4.0, precision="f32", thermal=True, steps=100),
        # a batch of uneven pore replicas with an ellipsoid each, and the state of every replica
        dict(name="batch128_f32", kind="step", wall="batch", replicas=128, precision="f32",
             thermal=True, steps=100),
        # a smaller batch in FP64
        dict(name="batch32_f64", kind="step", wall="batch", replicas=32, precision="f64",
             thermal=True, steps=100),
        # ragged: odd sides, obstacles (rows with several fluid runs), one sphere
        dict(name="obstacles_odd_f32", kind="step", wall="obstacles", nx=45, ny=37, nz=61,
             bodies=1, radius=3.0, precision="f32", thermal=True, steps=100),
        # the reverse pass on a fixed sphere in uniform flow, 64^3, window of 200 steps
        dict(name="adjoint64_fixed_f32", kind="adjoint", nx=64, ny=64, nz=64, radius=4.0,
             fixed=True, precision="f32", thermal=False, window=200, every=20),
        # and through the rigid-body integrator of a free sphere in a thermal fluid, FP64, odd box
        dict(name="adjoint_free_f64", kind="adjoint", nx=43, ny=35, nz=51, radius=3.0,
             fixed=False, precision="f64", thermal=True, window=60, every=8),
        # a recorded trajectory: 32 bodies, 20,000 frames, 1000 lags, 8 radial bins
        dict(name="analysis_32x20000", kind="analysis", bodies=32, frames=20000, lags=1000, bins=8),
        # the paper's 15 ellipsoids of revolution, outer and inner shells together
        dict(name="construct_30", kind="construct", ellipsoids=15, radius=4.25, steps=2000),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["resistance", "adjoint", "adjoint", "analysis", "analysis",
                                      "construct"])
    precision = rng.choice(["f32", "f32", "f64"])
    if kind == "resistance":
        return dict(kind=kind, nx=rng.randint(30, 72), radius=round(rng.uniform(2.0, 6.0), 2),
                    samples=rng.randint(3, 20))
    if kind == "adjoint":
        return dict(kind=kind, nx=rng.randint(24, 80), ny=rng.randint(24, 80),
                    nz=rng.randint(24, 80), radius=round(rng.uniform(2.0, 4.5), 2),
                    fixed=rng.random() < 0.5, precision=precision, thermal=rng.random() < 0.5,
                    window=_log(rng, 20, 200), every=rng.randint(1, 24))
    if kind == "analysis":
        frames = _log(rng, 300, 30000)
        return dict(kind=kind, bodies=_log(rng, 1, 48), frames=frames,
                    lags=min(frames - 1, _log(rng, 50, 1200)), bins=rng.randint(1, 12))
    if kind == "construct":
        return dict(kind=kind, ellipsoids=rng.randint(1, 24), radius=round(rng.uniform(2.0, 6.0), 2),
                    steps=_log(rng, 200, 2000))
    wall = rng.choice(["none", "none", "pore", "confined", "batch", "obstacles"])
    thermal = rng.random() < 0.8
    if wall == "batch":
        return dict(kind=kind, wall=wall, replicas=_log(rng, 4, 120 if precision == "f32" else 60),
                    precision=precision, thermal=True, steps=100)
    if wall == "confined":       # the pore beads need a wide box
        nx = rng.randint(76, 128)
        return dict(kind=kind, wall=wall, nx=nx, ny=nx, nz=rng.randint(64, 220),
                    bodies=rng.randint(1, 12), radius=3.5, precision=precision, thermal=True,
                    steps=rng.choice([50, 100]))
    lo, hi = (28, 72) if wall == "obstacles" else (24, 200)
    sides = [_log(rng, lo, hi) for _ in range(3)]
    if wall == "pore":
        sides[0] = sides[1] = max(32, sides[0])
    return dict(kind=kind, wall=wall, nx=sides[0], ny=sides[1], nz=sides[2],
                bodies=1 if min(sides) < 64 else rng.randint(1, 12),
                radius=round(rng.uniform(2.0, 4.0), 2), precision=precision, thermal=thermal,
                steps=rng.choice([7, 50, 100]))


# ------------------------------------------------------------------ inputs

def _placed(rng, n, reach, shape, pore=None):
    """n centres at random, `reach` apart (periodic), inside a pore along z when given."""
    L = np.array(shape, dtype=np.float64)
    out = []
    for _ in range(200000):
        if len(out) == n:
            break
        c = rng.uniform(0.0, 1.0, size=3) * L
        if pore is not None:
            d, th = rng.uniform(0.0, 1.0) * pore, rng.uniform(0.0, 2.0 * math.pi)
            c[:2] = L[:2] / 2.0 + d * np.array([math.cos(th), math.sin(th)])
        if all(np.linalg.norm((c - o) - L * np.round((c - o) / L)) > reach for o in out):
            out.append(c)
    return out


def _sphere(radius, pos, rng, gamma=W.GAMMA_FREE, **kw):
    m, inertia = W.solid_body_mass_inertia(1.0, radius, radius, radius)
    return W.body_record(W.sphere_beads(radius, W.sphere_bead_count(radius)), m, inertia, pos,
                         quat=W.random_quaternion(rng), gamma=gamma, **kw)


def workload(case, seed):
    """The simulation of a case as a record of paper_1604_01829_amd.workloads."""
    rng = np.random.default_rng([seed, 160401829])
    philox = int(rng.integers(1, 1 << 60))
    kT = KT if case.get("thermal") else 0.0
    if case["kind"] == "resistance":
        wl = W.stokes_flow_workload(L=case["nx"], radius=case["radius"])
        wl["replicas"][0]["bodies"][0]["pos"] = case["nx"] / 2.0 + rng.uniform(-0.5, 0.5, size=3)
        return wl
    if case["kind"] == "adjoint":
        shape = (case["nx"], case["ny"], case["nz"])
        body = _sphere(case["radius"], np.array(shape) / 2.0 + rng.uniform(-0.5, 0.5, size=3), rng,
                       gamma=W.GAMMA_FIXED if case["fixed"] else W.GAMMA_FREE, fixed=case["fixed"],
                       omega=(0.002, -0.001, 0.0015))
        return dict(precision=case["precision"], params=W.default_params(kT=kT, u0=(0.01, 0.0, 0.0)),
                    replicas=[dict(shape=shape, seed=philox, mask=None, bodies=[body])])
    if case["wall"] == "batch":
        reps = []
        sides = np.random.default_rng(case["replicas"]).choice([32, 40, 48, 56, 64], case["replicas"])
        for r, L in enumerate(sides.tolist()):
            pore, phi = 0.4 * L, rng.uniform(1.0, 4.0)
            b = 0.1 * L / phi ** (1.0 / 3.0)
            a = phi * b
            m, inertia = W.solid_body_mass_inertia(1.0, a, b, b)
            pos = _placed(rng, 1, 0.0, (L, L, L), 0.5 * max(0.0, pore - a - 2.0))[0]
            reps.append(dict(shape=(L, L, L), seed=philox + r, mask=W.pore_mask(L, L, L, pore),
                             bodies=[W.body_record(W.ellipsoid_beads(a, b, b), m, inertia, pos,
                                                   quat=W.random_quaternion(rng),
                                                   gamma=W.GAMMA_FREE)]))
        return dict(precision=case["precision"], params=W.default_params(kT=kT), replicas=reps)
    nx, ny, nz = shape = (case["nx"], case["ny"], case["nz"])
    radius, mask, inside = case["radius"], None, None
    if case["wall"] in ("pore", "confined"):
        pore = 0.3125 * nx if case["wall"] == "confined" or nx >= 128 else 0.4 * nx
        mask, inside = W.pore_mask(nx, ny, nz, pore), max(0.0, pore - radius - 2.0)
    elif case["wall"] == "obstacles":    # a block and a plate with gaps around them
        mask = np.zeros((nz, ny, nx), dtype=np.uint8)
        mask[nz // 8:nz // 8 + 6, ny // 5:ny // 5 + 9, nx // 4:nx // 4 + 7] = 1
        mask[3 * nz // 4:3 * nz // 4 + 2, 3:ny - 3, nx // 3:nx - 4] = 1
    if case["wall"] == "none" and case["bodies"] > 1:   # ellipsoids, as in the 256^3 workload
        semi = [(4.0, 2.0), (8.0, 2.0), (8.0, 4.0), (2.0, 4.0)]
        bodies = []
        for k, pos in enumerate(_placed(rng, case["bodies"], 18.0, shape)):
            a, b = semi[k % 4]
            m, inertia = W.solid_body_mass_inertia(1.0, a, b, b)
            bodies.append(W.body_record(W.ellipsoid_beads(a, b, b), m, inertia, pos,
                                        quat=W.random_quaternion(rng), gamma=W.GAMMA_FREE))
    else:
        bodies = [_sphere(radius, pos, rng)
                  for pos in _placed(rng, case["bodies"], 2.0 * radius + 2.0, shape, inside)]
    params = W.default_params(kT=kT, g_ext=(0.0, 0.0, 0.0) if kT else (1e-5, 0.0, 0.0))
    rep = dict(shape=shape, seed=philox, mask=mask, bodies=bodies)
    if case["wall"] == "confined":
        params.update(md_substeps=2, wca_epsilon=KT)
        rep["wall_sites"] = (W.pore_wall_sites(nx, ny, nz, pore), W.PORE_SITE_RADIUS)
        for b in bodies:
            b["ev"] = (W.inner_layer_sphere(radius), W.INNER_LAYER_RADIUS)
    return dict(precision=case["precision"], params=params, replicas=[rep])


def trajectory(case, seed):
    """Poses [frames, bodies, 7]: random walks about a pore axis, random small rotations."""
    F, B = case["frames"], case["bodies"]
    g = torch.Generator(device=DEVICE).manual_seed(seed)
    n = dict(generator=g, device=DEVICE, dtype=torch.float64)
    r, th = 2.0 + 22.0 * torch.rand(B, **n), 2.0 * math.pi * torch.rand(B, **n)
    steps = 0.05 * torch.randn(F, B, 3, **n)
    steps[0] = torch.stack([64.0 + r * th.cos(), 64.0 + r * th.sin(), 0.0 * r], dim=1)
    v = 0.03 * torch.randn(F, B, 3, **n)
    ang = v.norm(dim=2, keepdim=True)
    q = torch.cat([(ang / 2).cos(), (ang / 2).sin() * v / ang], dim=2)
    q[0] = torch.randn(B, 4, **n)
    q[0] /= q[0].norm(dim=1, keepdim=True)
    k = 1
    while k < F:                        # prefix products of the rotations
        q = torch.cat([q[:k], _qmul(q[:-k], q[k:])], dim=0)
        k *= 2
    return torch.cat([steps.cumsum(0), q / q.norm(dim=2, keepdim=True)], dim=2).contiguous()


def _separated(ax, n, rng):
    """n points at random on an ellipsoid, at least 3/4 of the mean spacing apart (less where
    they do not fit), as C.separated_shell places them: a candidate is kept if no kept point is
    near."""
    u = rng.normal(size=(100 * n, 3))
    u /= np.linalg.norm(u, axis=1, keepdims=True)
    area = np.linalg.norm(u * np.prod(ax) / ax, axis=1)
    p = (ax * u)[rng.uniform(size=len(u)) * area.max() < area]
    gap = 0.75 * math.sqrt(W.ellipsoid_area(*ax) / n)
    while True:
        kept = p[:1]
        for block in np.split(p[1:], range(256, len(p) - 1, 256)):
            far = ((block[:, None] - kept[None]) ** 2).sum(2).min(1) >= gap * gap
            fresh = []
            for x in block[far]:
                if all((x[0] - y[0]) ** 2 + (x[1] - y[1]) ** 2 + (x[2] - y[2]) ** 2 >= gap * gap
                       for y in fresh):
                    fresh.append(x)
            if fresh:
                kept = np.concatenate([kept, fresh])
            if len(kept) >= n:
                return kept[:n]
        gap *= 0.9


def shells(case, seed):
    """Semi-axes and starting beads of the outer and inner shells of ellipsoids of revolution."""
    rng = np.random.default_rng([seed, 21])
    phis = [1 / 10, 1 / 5, 1 / 4, 1 / 3, 1 / 2, 2 / 3, 4 / 5, 9 / 10, 10 / 9, 5 / 4, 3 / 2, 2, 4, 5, 10]
    axes, start = [], []
    for k in range(case["ellipsoids"]):
        phi = phis[k % 15]
        b = (case["radius"] ** 3 / phi) ** (1 / 3)
        for d in (0.0, 0.5):
            ax = np.maximum(np.array([phi * b - d, b - d, b - d]), 0.3)
            axes.append(tuple(ax))
            start.append(_separated(ax, C.shell_count(*ax), rng))
    return axes, start


def prepare(case, seed):
    state = dict(case=dict(case))
    if case["kind"] == "analysis":
        state["traj"] = trajectory(case, seed)
        state["ref"] = np.tile([1.0, 0.0, 0.0], (case["bodies"], 1))
        state["edges"] = np.linspace(0.0, 32.0, case["bins"] + 1)
        return state
    if case["kind"] == "construct":
        state["axes"], state["start"] = shells(case, seed)
        return state
    wl = workload(case, seed)
    sim = state["sim"] = lbrb.simulation_from_workload(wl, device=DEVICE)
    sizes = [4 * int(np.prod(r["shape"])) for r in wl["replicas"]]
    state["fields"] = torch.empty(sum(sizes), dtype=sim.dtype, device=DEVICE)
    state["starts"] = np.concatenate([[0], np.cumsum(sizes)]).tolist()
    if case["kind"] == "adjoint":
        state["weights"] = _weights(case)
    if case["kind"] == "resistance":
        state["u"] = wl["replicas"][0]["walls"][1]
    sim.step(WARM)
    return state


def _weights(case):
    w = np.zeros((case["window"], 1, 3))     # the window's mean drag along x
    w[:, 0, 0] = 1.0 / case["window"]
    return w


# ------------------------------------------------------------------ one pass

def _read(state):
    """The state a program records: poses, motion, forces of every body, density and velocity of
    every node (forces in the context's precision)."""
    sim, f = state["sim"], state["fields"]
    bodies, totals = [], []
    for r in range(len(sim.shapes)):
        at = f.data_ptr() + state["starts"][r] * f.element_size()
        _, t, bs = lbrb.lb_observables(sim.ctx, r, sim.n_bodies[r], at)
        bodies += bs
        totals.append([t.mass])
    motion = np.array([b.pos[:] + b.quat[:] for b in bodies])
    force = np.array([b.force[:] + b.torque[:] for b in bodies])
    return dict(mass=np.array(totals), motion=motion, fields=f,
                force=force.astype(np.float32 if sim.f32 else np.float64))


def run(state):
    case = state["case"]
    if case["kind"] == "analysis":
        t, lags = state["traj"], case["lags"]
        lab, body = A.lab_frame(t), A.body_frame(t)
        pore, radial = A.pore_frame(t, (64.0, 64.0))
        sums, counts = A.binned_msd(pore, radial, state["edges"], lags)
        return dict(lab=lab, body=body, pore=pore, radial=radial, msd_lab=A.msd(lab, lags),
                    msd_body=A.msd(body, lags), msd_rot=A.rotation_msd(t, state["ref"], lags),
                    sums=sums, counts=counts)
    if case["kind"] == "construct":
        p, v = C.relax_shells(state["axes"], state["start"], n_steps=case["steps"], device=DEVICE)
        return dict(positions=np.concatenate(p), velocities=np.concatenate(v))
    sim = state["sim"]
    if case["kind"] == "adjoint":
        J, dg, do = sim.adjoint(case["window"], state["weights"], case["every"])
        real = np.float32 if sim.f32 else np.float64    # the parameters an optimiser holds
        return dict(J=np.array([J], real), dgamma=dg.astype(real), doffsets=do.astype(real))
    if case["kind"] == "resistance":
        F, xi = lbrb.stokes_flow_resistance(sim, 0, 0, state["u"], 0, case["samples"], 10)
        return dict(_read(state), drag=F, xi=xi)
    sim.step(case["steps"])
    return _read(state)


# ------------------------------------------------------------------ what a pass needs

def _fluid(case):
    """(nodes, fluid nodes) of a case's boxes, about."""
    if case.get("wall") == "batch":      # mean over the sides
        n = case["replicas"] * np.mean([s ** 3 for s in (32, 40, 48, 56, 64)])
        return n, n * math.pi * 0.16
    nx = case["nx"]
    n = nx * case.get("ny", nx) * case.get("nz", nx)
    if case.get("wall") in ("pore", "confined"):
        f = 0.3125 if case["wall"] == "confined" or nx >= 128 else 0.4
        return n, n * math.pi * f * f
    return n, n


def work(case):
    if case["kind"] == "analysis":
        F, B, lags = case["frames"], case["bodies"], case["lags"]
        pairs = B * (lags * F - lags * (lags + 1) / 2)
        series = 8.0 * F * B * (3 + 6 + 3 + 1)
        # squared increments of 3 + 6 + 3 components, a dot product and an arccosine
        return dict(bytes=56.0 * F * B * 4 + 2 * series, flops=pairs * (12 * 3 + 5 + 25))
    if case["kind"] == "construct":
        beads = 2.0 * case["ellipsoids"] * 4 * math.pi * case["radius"] ** 2
        return dict(bytes=96.0 * beads, flops=case["steps"] * beads * (18 * 20 + 60))
    n, fluid = _fluid(case)
    real = 4 if case.get("precision") == "f32" else 8
    step = 2 * 19 * real * fluid
    if case["kind"] == "adjoint":
        T, K = case["window"], min(case["window"], case["every"])
        # forward, checkpoints, recomputed steps, reverse steps (state and adjoint in, adjoint out)
        back = 3 * 19 * real * fluid
        return dict(bytes=T * step + step * -(-T // K) + (T - -(-T // K)) * step + T * back,
                    flops=T * fluid * (250 * 2 + 600.0))
    steps = case["samples"] * 10 if case["kind"] == "resistance" else case["steps"]
    return dict(bytes=float(steps * step + 19 * real * fluid + 4 * real * n),
                flops=steps * fluid * 250.0)


# ------------------------------------------------------------------ the same in plain FP64

CV = np.array([(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
               (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
               (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)])
WT = np.array([1 / 3] + [1 / 18] * 6 + [1 / 36] * 12)
OPP = [0] + [i + 1 if i % 2 else i - 1 for i in range(1, 19)]


def _basis():
    x, y, z = (CV[:, a].astype(np.float64) for a in range(3))
    c2 = x * x + y * y + z * z
    return np.stack([1 + 0 * x, x, y, z, c2 - 1, 3 * x * x - c2, y * y - z * z, x * y, y * z, z * x,
                     (3 * c2 - 5) * x, (3 * c2 - 5) * y, (3 * c2 - 5) * z, (y * y - z * z) * x,
                     (z * z - x * x) * y, (x * x - y * y) * z, 3 * c2 * c2 - 6 * c2 + 1,
                     (2 * c2 - 3) * (3 * x * x - c2), (2 * c2 - 3) * (y * y - z * z)])


def _dev(a):
    return torch.as_tensor(np.asarray(a), dtype=torch.float64, device=DEVICE)


def _philox(step, index, domain, block, seed):
    """Philox4x32-10 words of counter (step low, index, domain << 16 | block, step high)."""
    M = 0xFFFFFFFF
    c = [torch.full_like(index, step & M), index.clone(),
         torch.full_like(index, (domain << 16) | block), torch.full_like(index, step >> 32)]
    k0, k1 = seed & M, (seed >> 32) & M

    def mul(a, b):      # high and low words of a product
        lo, hi = a * (b & 0xFFFF), a * (b >> 16)
        return (hi + (lo >> 16)) >> 16, (lo + ((hi & 0xFFFF) << 16)) & M

    for _ in range(10):
        h0, l0 = mul(0xD2511F53, c[0])
        h1, l1 = mul(0xCD9E8D57, c[2])
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & M, (k1 + 0xBB67AE85) & M
    return c


def _half(w, high):
    return (2.0 * ((w >> 16 if high else w) & 0xFFFF) + 1.0 - 65536.0) / 131072.0


def _qmul(a, b):
    w, x, y, z = a.unbind(-1)
    e, f, g, h = b.unbind(-1)
    return torch.stack([w * e - x * f - y * g - z * h, w * f + x * e + y * h - z * g,
                        w * g - x * h + y * e + z * f, w * h + x * g - y * f + z * e], dim=-1)


def _matrix(q):
    w, x, y, z = q.unbind(-1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)],
                       dim=-1).reshape(*q.shape[:-1], 3, 3)


class Reference:
    """One box of a workload record stepped in plain torch FP64 (differentiable)."""

    def __init__(self, wl):
        p, rep = wl["params"], wl["replicas"][0]
        self.shape = nx, ny, nz = rep["shape"]
        self.seed, self.kT, self.step_no = int(rep["seed"]), p["kT"], 0
        self.L = _dev([nx, ny, nz])
        self.g = _dev(p["g_ext"])
        self.rho0 = p["rho0"]
        E = _basis()
        b = (E * E * WT).sum(1)
        rate = [0.0] * 4 + [p["tau_bulk"]] + [p["tau_shear"]] * 5 + [p["tau_odd"]] * 6 + [p["tau_even"]] * 3
        gam = np.array([0.0 if t == 0.0 else 1.0 - 1.0 / t for t in rate])
        self.gam, self.E, self.back = _dev(gam)[:, None], _dev(E), _dev(E.T * WT[:, None] / b)
        self.amp = _dev(np.sqrt(12.0 * 3.0 * self.kT * self.rho0 * b * (1 - gam ** 2)))[4:, None]
        mask = rep["mask"]
        self.solid = None if mask is None else torch.as_tensor(np.asarray(mask) != 0, device=DEVICE)
        self.from_wall, self.fluid = [None] * 19, None
        if mask is not None:
            self.fluid = (~self.solid).reshape(-1)
            u = np.zeros((256, 3))
            for k, v in (rep.get("walls") or {}).items():
                u[k] = v
            uw = _dev(u)[torch.as_tensor(np.asarray(mask, np.int64), device=DEVICE)]
            for i in range(1, 19):
                at = self._shift(self.solid, i)
                add = 6 * WT[i] * self.rho0 * (self._shift(uw, i) @ _dev(CV[i]))
                self.from_wall[i] = (at, add)
        u0 = np.array(p["u0"])
        cu = CV @ u0
        f0 = WT * self.rho0 * (3 * cu + 4.5 * cu ** 2 - 1.5 * (u0 @ u0))
        self.f = _dev(f0)[:, None, None, None].expand(19, nz, ny, nx).contiguous()
        self.dense = torch.arange(nx * ny * nz, device=DEVICE)
        # bodies, as arrays over bodies and beads
        bs = rep["bodies"]
        self.m = max(1, int(p.get("md_substeps", 0)))
        self.dt = 1.0 / self.m
        self.body = torch.as_tensor(np.repeat(np.arange(len(bs)), [len(b["offsets"]) for b in bs]),
                                    device=DEVICE)
        self.off = _dev(np.concatenate([b["offsets"] for b in bs]))
        self.gamma = _dev([b["gamma"] for b in bs])
        self.mass, self.inertia = _dev([b["mass"] for b in bs])[:, None], _dev([b["inertia"] for b in bs])
        self.free = _dev([0.0 if b["fixed"] else 1.0 for b in bs])[:, None]
        self.R, self.q = _dev([b["pos"] for b in bs]), _dev([b["quat"] / np.linalg.norm(b["quat"]) for b in bs])
        self.V, self.w = _dev([b["vel"] for b in bs]) * self.free, _dev([b["omega"] for b in bs]) * self.free
        self.F, self.T = torch.zeros_like(self.R), torch.zeros_like(self.R)
        self.eps = p.get("wca_epsilon", 0.0)
        if self.eps:
            self.ev = _dev(np.concatenate([b["ev"][0] for b in bs]))
            self.ev_body = torch.as_tensor(np.repeat(np.arange(len(bs)), [len(b["ev"][0]) for b in bs]),
                                           device=DEVICE)
            self.ev_radius = float(bs[0]["ev"][1])
            self.reach = float(np.linalg.norm(bs[0]["ev"][0], axis=1).max())
            self.sites, self.site_radius = _dev(rep["wall_sites"][0]), float(rep["wall_sites"][1])

    @staticmethod
    def _shift(a, i):
        return torch.roll(a, shifts=(int(CV[i][2]), int(CV[i][1]), int(CV[i][0])), dims=(0, 1, 2))

    def streamed(self):
        out = []
        for i in range(19):
            d = self._shift(self.f[i], i)
            if self.from_wall[i] is not None:
                at, add = self.from_wall[i]
                d = torch.where(at, self.f[OPP[i]] + add, d)
            out.append(d)
        return torch.stack(out).reshape(19, -1)

    def velocity(self, d):
        drho = d.sum(0)
        j = _dev(CV.T) @ d
        return self.rho0 + drho, (j + 0.5 * self.g[:, None]) / (self.rho0 + drho)

    def half_kick(self, w, T):
        return w + 0.5 * self.dt * (T - torch.cross(w, self.inertia * w, dim=1)) / self.inertia * self.free

    def wca(self, R, rot):
        """Force and torque of the excluded volume on every body."""
        arm = (rot[self.ev_body] @ self.ev[:, :, None])[:, :, 0]
        x = R[self.ev_body] + arm
        F = torch.zeros_like(x)

        def add(rows, other, sigma):
            d = x[rows][:, None] - other[None]
            d = d - self.L * torch.round(d / self.L)
            r2 = (d * d).sum(2)
            s6 = (sigma * sigma / r2) ** 3
            c = torch.where(r2 < 2 ** (1 / 3) * sigma * sigma, 24 * self.eps * (2 * s6 * s6 - s6) / r2, 0.0)
            F[rows] += (c[:, :, None] * d).sum(1)

        axis = (x[:, :2] - self.L[:2] / 2).norm(dim=1)     # only sites near the pore beads' ring
        ring = (self.sites[0, :2] - self.L[:2] / 2).norm()
        near = torch.nonzero(axis > ring - 1.13 * (self.ev_radius + self.site_radius))[:, 0]
        if len(near):
            add(near, self.sites, self.ev_radius + self.site_radius)
        d = R[:, None] - R[None]
        d = (d - self.L * torch.round(d / self.L)).norm(dim=2).cpu().numpy()
        for b, o in zip(*np.nonzero(d < 2 * self.reach + 1.13 * 2 * self.ev_radius)):
            if b != o:
                add(torch.nonzero(self.ev_body == int(b))[:, 0], x[self.ev_body == int(o)], 2 * self.ev_radius)
        z = torch.zeros_like(R)
        return z.index_add(0, self.ev_body, F), z.index_add(0, self.ev_body, torch.cross(arm, F, dim=1))

    def md_step(self, k, u, spread):
        dt, free = self.dt, self.free
        V = self.V + 0.5 * dt * self.F / self.mass * free
        w = self.half_kick(self.w, self.T)
        R, q = self.R + dt * V, self.q
        if bool(free.any()) and bool((w.detach() != 0).any()):
            wn = w.norm(dim=1, keepdim=True).clamp_min(1e-300)
            p = torch.cat([torch.cos(0.5 * dt * wn), torch.sin(0.5 * dt * wn) * w / wn], dim=1)
            q = _qmul(q, p)
            q = q / q.norm(dim=1, keepdim=True)
        rot = _matrix(q)
        wl = (rot @ w[:, :, None])[:, :, 0]
        arm = (rot[self.body] @ self.off[:, :, None])[:, :, 0]
        r = R[self.body] + arm
        v = (V[self.body] + torch.cross(wl[self.body], arm, dim=1)) * free[self.body]
        # trilinear stencil
        nx, ny, nz = self.shape
        base = torch.floor(r.detach() - 0.5)
        fr, i0 = r - 0.5 - base, base.long()
        idx, wt = [], []
        for c in range(8):
            o = (c & 1, (c >> 1) & 1, c >> 2)
            n = [(i0[:, a] + o[a]) % (nx, ny, nz)[a] for a in range(3)]
            idx.append(n[0] + nx * (n[1] + ny * n[2]))
            wt.append(math.prod(fr[:, a] if o[a] else 1.0 - fr[:, a] for a in range(3)))
        idx, wt = torch.stack(idx, 1), torch.stack(wt, 1)
        if self.fluid is not None:
            wt = wt * self.fluid[idx]
        uk = (wt[None] * u[:, idx]).sum(2).T
        gam = self.gamma[self.body][:, None]
        F = -gam * (v - uk)
        if self.kT > 0:
            b = _philox(self.step_no, torch.arange(len(r), device=DEVICE), 1, k, self.seed)
            xi = torch.stack([_half(b[0], False), _half(b[0], True), _half(b[1], False)], dim=1)
            F = F + torch.sqrt(24.0 * self.kT * gam / dt) * xi
        spread = spread.index_add(1, idx.reshape(-1),
                                  -dt * (wt[:, :, None] * F[:, None]).reshape(-1, 3).T)
        z = torch.zeros_like(R)
        Fb = z.index_add(0, self.body, F)
        Tb = z.index_add(0, self.body, torch.cross(arm, F, dim=1))
        if self.eps:
            Fw, Tw = self.wca(R, rot)
            Fb, Tb = Fb + Fw, Tb + Tw
        Tb = (rot.transpose(1, 2) @ Tb[:, :, None])[:, :, 0]
        self.R, self.q, self.F, self.T = R, q, Fb, Tb
        self.V = V + 0.5 * dt * Fb / self.mass * free
        self.w = self.half_kick(w, Tb)
        return spread

    def step(self):
        d = self.streamed()
        rho, u0 = self.velocity(d)
        if self.fluid is not None:
            u0 = u0 * self.fluid
        spread = torch.zeros_like(u0)
        for k in range(self.m):
            spread = self.md_step(k, u0, spread)
        F = spread + self.g[:, None]
        m = self.E @ d
        u = (m[1:4] + 0.5 * F) / rho
        x, y, z = u
        X, Y, Z = F
        eq = rho * torch.stack([x * x + y * y + z * z, 2 * x * x - y * y - z * z, y * y - z * z,
                                x * y, y * z, z * x])
        src = torch.stack([2 * (x * X + y * Y + z * Z), 2 * (2 * x * X - y * Y - z * Z),
                           2 * (y * Y - z * Z), x * Y + y * X, y * Z + z * Y, z * X + x * Z])
        gm = self.gam[4:10]
        new = [m[:1], m[1:4] + F, eq + gm * (m[4:10] - eq) + 0.5 * (1 + gm) * src,
               self.gam[10:] * m[10:]]
        m = torch.cat(new)
        if self.kT > 0:
            words = [w for blk in (0, 1) for w in _philox(self.step_no, self.dense, 0, blk, self.seed)]
            for h in range(15):
                m[4 + h] += self.amp[h] * _half(words[h >> 1], bool(h & 1))
        f = self.back @ m
        if self.fluid is not None:
            f = f * self.fluid
        nx, ny, nz = self.shape
        self.f = f.reshape(19, nz, ny, nx)
        self.step_no += 1

    def read(self, real):
        d = self.streamed()
        rho, u = self.velocity(d)
        f = torch.cat([rho[None], u])
        n = f.shape[1]
        mass = d.sum() if self.fluid is None else (d.sum(0) * self.fluid).sum()
        if self.fluid is not None:
            f, n = f * self.fluid, self.fluid.sum()
        return dict(mass=(mass + n * self.rho0).reshape(1, 1).cpu().numpy(),
                    motion=torch.cat([self.R, self.q], dim=1), fields=f.T.reshape(-1),
                    force=torch.cat([self.F, self.T], dim=1))


def _exact_simulation(case, seed):
    ref = Reference(workload(case, seed))
    with torch.no_grad():
        for _ in range(WARM):
            ref.step()
    if case["kind"] == "adjoint":
        ref.gamma.requires_grad_(True)
        ref.off.requires_grad_(True)
        J = 0.0
        for _ in range(case["window"]):
            ref.step()
            J = J + ref.F[0, 0] / case["window"]
        dg, do = torch.autograd.grad(J, [ref.gamma, ref.off])
        return dict(J=J.detach().reshape(1), dgamma=dg, doffsets=do)
    with torch.no_grad():
        if case["kind"] == "resistance":
            drag = torch.zeros(3, dtype=torch.float64, device=DEVICE)
            for _ in range(case["samples"]):
                for _ in range(10):
                    ref.step()
                drag += ref.F[0] / case["samples"]
            u = _dev([0.0, 0.0, W.STOKES_U_PAPER])
            return dict(ref.read(case), drag=drag, xi=float(drag @ u / (u @ u)))
        for _ in range(case["steps"]):
            ref.step()
        return ref.read(case)


def _exact_analysis(case, seed):
    t = trajectory(case, seed)
    lags, edges = case["lags"], np.linspace(0.0, 32.0, case["bins"] + 1)
    x, rot = t[:, :, :3], _matrix(t[:, :, 3:])
    dx, A0, A1 = x[1:] - x[:-1], rot[:-1], rot[1:]
    rel = A0.transpose(2, 3) @ A1             # columns: the body axes in the frame one step before
    ang = torch.stack([torch.atan(rel[..., 1, 2] / rel[..., 2, 2]),
                       torch.atan(rel[..., 2, 0] / rel[..., 0, 0]),
                       torch.atan(rel[..., 0, 1] / rel[..., 1, 1])], dim=2)
    th = torch.atan2(x[:-1, :, 1] - 64.0, x[:-1, :, 0] - 64.0)
    c, s = th.cos(), th.sin()
    dp = torch.stack([c * dx[..., 0] + s * dx[..., 1], c * dx[..., 1] - s * dx[..., 0], dx[..., 2]], dim=2)

    def series(d):
        return torch.cat([torch.zeros_like(d[:1]), d.cumsum(0)]).transpose(0, 1).contiguous()

    lab = (x - x[:1]).transpose(0, 1).contiguous()
    body = series(torch.cat([(A0.transpose(2, 3) @ dx[..., None])[..., 0], ang], dim=2))
    pore = series(dp)
    radial = torch.hypot(x[..., 0] - 64.0, x[..., 1] - 64.0).T.contiguous()
    p = rot[..., 0].transpose(0, 1).contiguous()
    e = _dev(edges)
    onehot = ((radial[None] >= e[:-1, None, None]) & (radial[None] < e[1:, None, None])).double()
    out = dict(msd_lab=[], msd_body=[], msd_rot=[], sums=[], counts=[])
    for k in range(1, lags + 1):
        out["msd_lab"].append(((lab[:, k:] - lab[:, :-k]) ** 2).mean(1))
        out["msd_body"].append(((body[:, k:] - body[:, :-k]) ** 2).mean(1))
        cos = (p[:, k:] * p[:, :-k]).sum(2).clamp(-1.0, 1.0)
        out["msd_rot"].append((torch.acos(cos) ** 2).mean(1))
        h = onehot[:, :, :-k].reshape(case["bins"], -1)
        out["sums"].append(h @ ((pore[:, k:] - pore[:, :-k]) ** 2).reshape(-1, 3))
        out["counts"].append(h.sum(1))
    return dict({n: torch.stack(v, dim=1).contiguous() for n, v in out.items()}, lab=lab, body=body,
                pore=pore, radial=radial)


def _exact_construct(case, seed):
    axes, start = shells(case, seed)
    counts = [len(s) for s in start]
    S, n = len(counts), max(counts)
    here = torch.arange(n, device=DEVICE)[None] < torch.as_tensor(counts, device=DEVICE)[:, None]
    x = torch.zeros(S, n, 3, dtype=torch.float64, device=DEVICE)
    x[here] = _dev(np.concatenate(start))
    v = torch.zeros_like(x)
    P = C.DEFAULT_PARAMS
    a = _dev(axes)[:, None]
    a2, amax = a * a, a.amax(2)
    both = here[:, :, None] & here[:, None, :] & ~torch.eye(n, dtype=torch.bool, device=DEVICE)
    s2, g = P["sigma"] ** 2, 0.5 * P["damping"] * P["dt"]
    lo, hi = (-a2.amin(2)).expand(S, n), amax * x.norm(dim=2) + 1.0
    for _ in range(200):                      # the closest surface point's parameter, by bisection
        t = 0.5 * (lo + hi)
        big = ((x * a / (t[..., None] + a2)) ** 2).sum(2) > 1.0
        lo, hi = torch.where(big, t, lo), torch.where(big, hi, t)
    for _ in range(case["steps"]):
        d = x[:, :, None] - x[:, None]
        r2 = (d * d).sum(3)
        u6 = (s2 / r2) ** 3
        coef = torch.where(both & (r2 < 2 ** (1 / 3) * s2), 24 * P["epsilon"] * (2 * u6 * u6 - u6) / r2, 0.0)
        F = (coef[..., None] * d).sum(2)
        for _ in range(5):                    # and then by Newton from the step before
            y = (x * a / (t[..., None] + a2)) ** 2
            Sm, dS = y.sum(2), -2.0 * (y / (t[..., None] + a2)).sum(2)
            rs = Sm.rsqrt()
            t = torch.where(here, t + 2.0 * (rs - 1.0) * Sm / (rs * dS), t)
        F = F - 2.0 * P["k_surface"] * (x - x * a2 / (t[..., None] + a2))
        v = torch.where(here[..., None], ((1.0 - g) * v + P["dt"] * F / P["mass"]) / (1.0 + g), v)
        x = x + P["dt"] * v
    return dict(positions=x[here], velocities=v[here])


def exact(case, seed):
    if case["kind"] == "analysis":
        return _exact_analysis(case, seed)
    if case["kind"] == "construct":
        return _exact_construct(case, seed)
    if case.get("wall") == "batch":
        return None                           # a box at a time takes minutes
    return _exact_simulation(case, seed)
