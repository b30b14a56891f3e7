"""Moving walls on the GPU against the oracle, and the Stokes-flow resistance protocol.

- parity: a box with wall ids moving in different directions (one id at rest) around a fixed
  and a free sphere, and a pore whose wall slides along its axis, thermal and deterministic,
  FP64 and FP32, eager and graph-replayed steps, and batched replicas with different wall
  velocities, element by element against the oracle (tolerances of the other parity tests:
  1e-11 of the field scale in FP64, 1e-5 in FP32);
- plane Couette flow: the exact linear profile of unit relaxation rates on the GPU;
- lb_set_wall_velocity: argument, state and capacity errors; mask and velocity in either
  order; walls given zero velocity are plain walls, bit for bit;
- the Stokes-flow protocol (Sec. 2.3, eq. (stokesflow)): the GPU's mean bead force against
  the oracle running the same protocol, the resistance independent of the imposed velocity
  at small Reynolds number, and the paper-sized 50^3 channel (parity of its first steps,
  then the developed resistance).
"""
import math

import numpy as np
import pytest

from paper_1604_01829_amd import lbrb
from paper_1604_01829_amd import workloads as W
from tests.helpers import (compare, gpu_from_workload, oracle_from_workload,
                           oracle_stokes_resistance)
from tests.test_gpu_parity import _assert_close, _print, pore_case

pytestmark = pytest.mark.gpu

U = 0.01


def walls_case(precision, kT, velocities=None, seed=4242):
    """12 x 14 x 10 box: wall 1 on the y = 0 face, wall 2 on the y = 13 face, wall 3 on the
    z = 0 face, wall 5 on the x = 0 face, wall 4 (at rest) filling x = 11 of the upper half;
    a fixed sphere R = 2 and a free sphere R = 1.5 clear of the walls."""
    nx, ny, nz = 12, 14, 10
    mask = np.zeros((nz, ny, nx), np.uint8)
    mask[:, :, 0] = 5
    mask[:, :, nx - 1][:, ny // 2:] = 4
    mask[:, 0, :] = 1
    mask[:, ny - 1, :] = 2
    mask[0, :, :] = 3
    if velocities is None:
        velocities = {1: (0.0, 0.0, U), 2: (0.5 * U, 0.0, -U), 3: (U / 3, -U / 4, 0.0),
                      5: (0.0, 0.5 * U, U / 3)}
    R1, R2 = 2.0, 1.5
    o1 = W.sphere_beads(R1, W.sphere_bead_count(R1))
    o2 = W.sphere_beads(R2, W.sphere_bead_count(R2))
    m1, I1 = W.solid_body_mass_inertia(1.0, R1, R1, R1)
    m2, I2 = W.solid_body_mass_inertia(1.0, R2, R2, R2)
    bodies = [W.body_record(o1, m1, I1, (6.3, 7.1, 5.4), gamma=W.GAMMA_FIXED, fixed=True),
              W.body_record(o2, m2, I2, (3.6, 4.2, 6.8), quat=(0.9, 0.1, -0.3, 0.2),
                            vel=(1e-3, -2e-3, 5e-4), omega=(2e-3, 0.0, -1e-3),
                            gamma=W.GAMMA_FREE)]
    return dict(name="walls", precision=precision, steps=40,
                params=W.default_params(kT=kT, g_ext=(1e-6, 0.0, 2e-6), tau_shear=0.8,
                                        tau_bulk=1.1, tau_odd=0.9, tau_even=1.2),
                replicas=[dict(shape=(nx, ny, nz), seed=seed, mask=mask, bodies=bodies,
                               walls=velocities)])


def _tol(precision):
    return (1e-11, 1e-13, 1e-12) if precision == "f64" else (1e-5, 1e-6, 1e-6)


def _run_and_compare(wl, precision, steps, graph=False, tag=""):
    gpu = gpu_from_workload(wl)
    if not graph:
        gpu.set_graph_steps(0)
    orc = oracle_from_workload(wl)
    done = 0
    for s in steps:
        gpu.step(s - done)
        orc.step(s - done)
        done = s
        e = compare(gpu, orc)
        _print(f"{tag} {precision} step {s}", e)
        _assert_close(e, *_tol(precision))
    return gpu, orc


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("kT", [0.0, 4e-5])
def test_moving_walls_box(precision, kT):
    wl = walls_case(precision, kT)
    gpu, orc = _run_and_compare(wl, precision, (1, 2, 7, 40), tag=f"walls kT={kT}")
    fb_g, fb_o = gpu.bead_forces(0, 0), orc.bead_forces(0)
    tol = 1e-11 if precision == "f64" else 1e-5
    assert np.abs(fb_g - fb_o).max() <= tol * np.abs(fb_o).max() + 1e-17
    # the pre-collision populations, element by element (zeros on boundary nodes)
    pg, pc = gpu.populations(0), orc.populations()
    assert np.abs(pg - pc).max() <= (1e-13 if precision == "f64" else 1e-6)


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_moving_walls_graph_replay(precision):
    wl = walls_case(precision, 4e-5)
    _run_and_compare(wl, precision, (100, 203), graph=True, tag="walls graph")


@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_sliding_pore_wall(precision):
    wl = pore_case(precision, 4e-5)
    wl["replicas"][0]["walls"] = {1: (0.0, 0.0, U)}
    _run_and_compare(wl, precision, (1, 3, 30), tag="sliding pore")


def test_batched_replicas_with_different_wall_velocities():
    a = walls_case("f64", 4e-5)
    b = walls_case("f64", 4e-5, velocities={1: (U, 0.0, 0.0), 2: (0.0, 0.0, 0.0),
                                            5: (0.0, -U, 0.0)}, seed=99)
    c = walls_case("f64", 4e-5, velocities={}, seed=7)
    wl = dict(a)
    wl["replicas"] = a["replicas"] + b["replicas"] + c["replicas"]
    gpu = gpu_from_workload(wl)
    gpu.set_graph_steps(4)
    gpu.step(9)
    for r in range(3):
        orc = oracle_from_workload(wl, r)
        orc.step(9)
        e = compare(gpu, orc, r)
        _print(f"batched replica {r}", e)
        _assert_close(e, *_tol("f64"))


def _couette_gpu(precision, steps):
    nx, ny, nz = 4, 18, 3
    mask = np.zeros((nz, ny, nx), np.uint8)
    mask[:, 0, :] = 1
    mask[:, ny - 1, :] = 2
    wl = dict(name="couette", precision=precision, steps=steps, params=W.default_params(),
              replicas=[dict(shape=(nx, ny, nz), seed=1, mask=mask, bodies=[],
                             walls={1: (-U, 0.0, 0.0), 2: (U, 0.0, 0.0)})])
    gpu = gpu_from_workload(wl)
    gpu.step(steps)
    return gpu.fields(0)


@pytest.mark.parametrize("precision,tol", [("f64", 1e-10), ("f32", 2e-4)])
def test_couette_profile_on_gpu(precision, tol):
    """All relaxation rates 1: the linear profile between walls halfway between boundary and
    fluid nodes is the exact steady state (pinned on the oracle).  FP32: one rounding of the
    shifted populations per step (~6e-8 of |f - w rho0|) over the ~1500-step diffusive time
    of the channel bounds the systematic error by ~1e-4 of U."""
    ny = 18
    f = _couette_gpu(precision, 6000)
    y = np.arange(1, ny - 1) + 0.5
    lin = -U + 2.0 * U * (y - 1.0) / (ny - 2)
    err = np.abs(f[:, 1:ny - 1, :, 1] - lin[None, :, None]).max()
    print(f"couette {precision}: max |u - linear| / U = {err / U:.3g}", flush=True)
    assert err <= tol * U
    assert np.abs(f[:, 1:ny - 1, :, 2:]).max() <= tol * U
    assert np.all(f[:, 0] == 0) and np.all(f[:, ny - 1] == 0)


def test_wall_velocity_errors_and_order():
    wl = walls_case("f64", 0.0)
    rep = wl["replicas"][0]
    need = lbrb.wall_link_bound(rep["mask"], rep["walls"])
    # capacity: too few links fails and changes nothing
    p = lbrb.make_params("f64", max_bodies=2, max_beads=400, max_wall_links=10,
                         **{k: v for k, v in wl["params"].items()})
    sim = lbrb.Simulation(p, lbrb.make_replicas([(rep["shape"], rep["seed"])]))
    sim.set_mask(0, rep["mask"])
    with pytest.raises(lbrb.LBError) as ei:
        sim.set_wall_velocity(0, 1, (0.0, 0.0, U))
    assert ei.value.code == lbrb.LB_ERR_CAPACITY
    sim.set_wall_velocity(0, 1, (0.0, 0.0, 0.0))           # no links: fits
    for bad in ((0, (0, 0, U)), (256, (0, 0, U)), (1, (math.nan, 0, 0))):
        with pytest.raises(lbrb.LBError) as ei:
            sim.set_wall_velocity(0, *bad)
        assert ei.value.code == lbrb.LB_ERR_ARG
    with pytest.raises(lbrb.LBError) as ei:
        sim.set_wall_velocity(1, 1, (0, 0, U))
    assert ei.value.code == lbrb.LB_ERR_ARG
    sim.step(1)
    with pytest.raises(lbrb.LBError) as ei:
        sim.set_wall_velocity(0, 2, (0, 0, U))
    assert ei.value.code == lbrb.LB_ERR_STATE
    sim.close()

    def run(order, velocities, mask):
        pp = lbrb.make_params("f64", max_bodies=2, max_beads=400, max_wall_links=need,
                              **{k: v for k, v in wl["params"].items()})
        s = lbrb.Simulation(pp, lbrb.make_replicas([(rep["shape"], rep["seed"])]))
        if order == "mask first":
            s.set_mask(0, mask)
        for k, u in velocities.items():
            s.set_wall_velocity(0, k, u)
        if order != "mask first":
            s.set_mask(0, mask)
        s.set_graph_steps(0)
        s.step(12)
        out = s.populations(0)
        s.close()
        return out

    a = run("mask first", rep["walls"], rep["mask"])
    b = run("velocities first", rep["walls"], rep["mask"])
    assert np.array_equal(a, b)
    # walls given zero velocity are plain walls
    ones = (rep["mask"] > 0).astype(np.uint8)
    c = run("mask first", {k: (0.0, 0.0, 0.0) for k in rep["walls"]}, rep["mask"])
    d = run("mask first", {}, ones)
    assert np.array_equal(c, d)


def _stokes_pair(precision, L, R, U_, tau, develop, samples, every):
    wl = W.stokes_flow_workload(L=L, radius=R, U=U_, tau_shear=tau, precision=precision)
    gpu = gpu_from_workload(wl)
    Fg, xg = lbrb.stokes_flow_resistance(gpu, 0, 0, (0, 0, U_), develop, samples, every)
    return wl, gpu, Fg, xg


@pytest.mark.parametrize("precision,tol", [("f64", 1e-10), ("f32", 1e-4)])
def test_stokes_protocol_matches_oracle(precision, tol):
    wl, gpu, Fg, xg = _stokes_pair(precision, 16, 2.5, 0.005, 1.0, 600, 100, 5)
    orc = oracle_from_workload(wl)
    Fo, xo = oracle_stokes_resistance(orc, 0, (0, 0, 0.005), 600, 100, 5)
    gross = float(np.linalg.norm(orc.bead_forces(0), axis=1).sum())
    print(f"stokes 16^3 {precision}: F_gpu={Fg} F_orc={Fo} xi={xg:.8g} ({xo:.8g})", flush=True)
    assert np.abs(Fg - Fo).max() <= tol * gross
    assert xo > 0 and abs(xg - xo) <= tol * gross / 0.005


def test_stokes_resistance_is_independent_of_the_velocity():
    """Stokes regime: the resistance does not depend on the imposed velocity or its sign.
    The nearly symmetric sphere at the channel centre makes the force odd in U up to the bead
    lattice's asymmetry, so what remains is of relative order Re^2 = (U R / nu)^2 <= 1.3e-5
    (the box is far smaller than the Oseen length nu / U ~ 800, so no O(Re) wake term)."""
    xi = {}
    for u in (1e-4, 2e-4, -1e-4):
        wl = W.stokes_flow_workload(L=20, radius=3.0, U=u, tau_shear=1.0, precision="f64")
        gpu = gpu_from_workload(wl)
        F, xi[u] = lbrb.stokes_flow_resistance(gpu, 0, 0, (0, 0, u), 3000, 100, 5)
        assert abs(F[0]) < 1e-2 * abs(F[2]) and abs(F[1]) < 1e-2 * abs(F[2])
        gpu.close()
    print("xi(U):", xi, flush=True)
    assert abs(xi[2e-4] / xi[1e-4] - 1) < 1e-4
    assert abs(xi[-1e-4] / xi[1e-4] - 1) < 1e-4


def test_stokes_paper_channel():
    """The paper's set-up: 50^3 box, walls on the +-y faces moving at 2.20 m/s along z,
    nu = 0.8 sigma^2/t0, sphere R = 5.25 nm.  The first steps match the oracle node by node;
    the developed resistance is stable, along the flow, and above the unbounded Stokes value
    6 pi nu rho R_h for any hydrodynamic radius the bead shell can have (R_h >= 0.8 R)."""
    wl = W.stokes_flow_workload(precision="f64")
    gpu = gpu_from_workload(wl)
    gpu.set_graph_steps(0)
    orc = oracle_from_workload(wl)
    gpu.step(4)
    orc.step(4)
    e = compare(gpu, orc)
    _print("stokes 50^3 step 4", e)
    _assert_close(e, *_tol("f64"))
    del orc
    gpu.set_graph_steps(100)
    u = (0.0, 0.0, W.STOKES_U_PAPER)
    F1, xi1 = lbrb.stokes_flow_resistance(gpu, 0, 0, u, 60000, 100, 10)
    F2, xi2 = lbrb.stokes_flow_resistance(gpu, 0, 0, u, 60000, 100, 10)
    nu = (W.STOKES_TAU_PAPER - 0.5) / 3.0
    stokes = 6 * math.pi * nu * 1.0 * 5.25
    print(f"stokes 50^3: xi = {xi1:.6g} then {xi2:.6g} (lattice units), "
          f"xi / (6 pi nu rho R) = {xi2 / stokes:.4f}", flush=True)
    assert abs(xi2 / xi1 - 1) < 1e-2
    assert xi2 > 0.8 * stokes and abs(F2[0]) < 1e-2 * F2[2] and abs(F2[1]) < 1e-2 * F2[2]


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_links_with_one_and_four_tiles_per_workgroup_agree_bitwise(precision):
    """The node update applies its tile's links itself, or leaves them to a launch."""
    import torch
    wl = W.stokes_flow_workload(L=22, radius=3.0, U=1e-3, precision=precision)
    out = []
    for tiles in (1, 4):
        sim = lbrb.simulation_from_workload(wl)
        sim.set_tuning(tiles_per_wg=tiles)
        sim.set_graph_steps(4)
        sim.step(11)
        out.append(sim.save_state())
        sim.close()
    assert torch.equal(out[0], out[1])


@pytest.mark.parametrize("precision", ["f32", "f64"])
@pytest.mark.parametrize("policy", [lbrb.LB_STORES_CACHED, lbrb.LB_STORES_STREAMING])
@pytest.mark.parametrize("holes", [False, True])
def test_links_after_either_store_and_before_the_mirror(holes, policy, precision):
    """The links that the node update adds to slots its workgroup has just stored, through the L2 or
    past it, against the launch after the update, bit for bit; and with a moving block between the
    fluid runs of a row, whose holes take the reflected populations with the links' terms in them."""
    import torch
    out = []
    for tiles in (1, 4):
        wl = walls_case(precision, 4e-5)
        if holes:
            wl["replicas"][0]["mask"][6:8, 2:4, 7:9] = 2
        sim = lbrb.simulation_from_workload(wl)
        sim.set_store_policy(policy)
        sim.set_tuning(tiles_per_wg=tiles)
        sim.set_graph_steps(4)
        sim.step(11)
        assert sim.tuned_settings()["streaming_stores"] == (policy == lbrb.LB_STORES_STREAMING)
        out.append((sim.save_state(), sim.populations()))
        sim.close()
    assert torch.equal(out[0][0], out[1][0])
    np.testing.assert_array_equal(out[0][1], out[1][1])
    orc = oracle_from_workload(wl)
    orc.step(11)
    gpu = lbrb.simulation_from_workload(wl)
    gpu.set_store_policy(policy)
    gpu.step(11)
    e = compare(gpu, orc)
    _print("links", e)
    _assert_close(e, *_tol(precision))
    gpu.close()
