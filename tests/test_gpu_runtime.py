"""GPU runtime behaviour through the C-ABI: graphs, determinism, checkpoints, batching of
uneven replicas, edge cases and error codes.  Parity cases compare with the FP64 oracle."""
import numpy as np
import pytest

from paper_1604_01829_amd import lbrb
from paper_1604_01829_amd import workloads as W
from tests.helpers import compare, gpu_from_workload, oracle_from_workload

pytestmark = pytest.mark.gpu


def _thermal_sphere(precision="f32"):
    wl = W.workload(1)
    wl["params"]["kT"] = 4e-5
    wl["precision"] = precision
    return wl


def _state_bytes(sim):
    return sim.save_state().cpu().numpy()


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_graph_replay_matches_eager_bitwise(precision):
    wl = _thermal_sphere(precision)
    a = gpu_from_workload(wl)
    a.set_graph_steps(0)
    b = gpu_from_workload(wl)
    b.set_graph_steps(20)
    a.step(47)
    b.step(47)   # two graph replays of 20 + 7 eager steps
    assert np.array_equal(_state_bytes(a), _state_bytes(b))
    a.step(40)
    b.step(40)   # graph of the other buffer parity
    assert np.array_equal(_state_bytes(a), _state_bytes(b))


def test_runs_are_deterministic():
    wl = pore_batch()
    a = gpu_from_workload(wl)
    b = gpu_from_workload(wl)
    a.step(25)
    b.step(25)
    assert np.array_equal(_state_bytes(a), _state_bytes(b))


def test_checkpoint_resume_is_bit_identical():
    wl = _thermal_sphere("f32")
    a = gpu_from_workload(wl)
    a.step(30)
    ck = a.save_state()
    a.step(30)
    end_a = _state_bytes(a)
    b = gpu_from_workload(wl)
    b.load_state(ck)
    b.step(30)
    assert np.array_equal(end_a, _state_bytes(b))
    t, bodies, _, rc = b.observables(0)
    assert t["step"] == 60 and rc == 0


def pore_batch():
    """Uneven replicas: three pores of different sides with one ellipsoid each, one periodic
    box with a sphere and one periodic box without bodies (ragged sizes)."""
    rng = np.random.default_rng(404)
    reps = []
    for k, L in enumerate((16, 20, 24)):
        phi = 1.5 + k
        req = 0.12 * L
        b = req / phi ** (1 / 3)
        a = phi * b
        offs = W.ellipsoid_beads(a, b, b)
        m, I = W.solid_body_mass_inertia(1.0, a, b, b)
        c = np.array([L / 2 + 0.7, L / 2 - 0.4, rng.uniform(0, L)])
        reps.append(dict(shape=(L, L, L + 3), seed=1000 + k, mask=W.pore_mask(L, L, L + 3, 0.4 * L),
                         bodies=[W.body_record(offs, m, I, c, quat=W.random_quaternion(rng),
                                               gamma=W.GAMMA_FREE)]))
    offs = W.sphere_beads(2.0, 35)
    m, I = W.solid_body_mass_inertia(1.0, 2.0, 2.0, 2.0)
    reps.append(dict(shape=(13, 11, 9), seed=77, mask=None,
                     bodies=[W.body_record(offs, m, I, (12.6, 0.3, 4.4), vel=(1e-3, 0, 0),
                                           gamma=W.GAMMA_FREE)]))
    reps.append(dict(shape=(33, 17, 5), seed=78, mask=None, bodies=[]))
    return dict(name="batch", precision="f32", steps=20,
                params=W.default_params(kT=4e-5, g_ext=(1e-6, 0.0, 3e-6)), replicas=reps)


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_batched_uneven_replicas_match_independent_oracles(precision):
    wl = pore_batch()
    wl["precision"] = precision
    gpu = gpu_from_workload(wl)
    gpu.set_graph_steps(0)
    orcs = [oracle_from_workload(wl, r) for r in range(len(wl["replicas"]))]
    for o in orcs:
        o.step(12)
    gpu.step(12)
    tol_u = 1e-11 if precision == "f64" else 1e-5
    tol_r = 1e-13 if precision == "f64" else 1e-6
    for r, o in enumerate(orcs):
        e = compare(gpu, o, r)
        print(f"replica {r} {precision}", {k: f"{v:.3g}" for k, v in e.items()
                                          if isinstance(v, float)}, flush=True)
        assert e["rc"] == 0 and e["solid_zero"] and e["finite"]
        assert e["rho"] <= tol_r
        assert e["u_abs"] <= tol_u * max(e["u_scale"], 1e-12)
        assert e["body_pos"] <= tol_r and e["body_quat"] <= tol_r


def test_batched_replica_equals_standalone_run():
    """A replica's trajectory does not depend on what it is batched with."""
    wl = pore_batch()
    batch = gpu_from_workload(wl)
    alone = gpu_from_workload(wl, replicas=[1])
    batch.step(15)
    alone.step(15)
    fb = batch.fields(1)
    fa = alone.fields(0)
    assert np.array_equal(fa, fb)
    assert np.array_equal(batch.observables(1)[1][0]["pos"], alone.observables(0)[1][0]["pos"])


def test_one_node_box_and_empty_replica():
    p = lbrb.make_params("f64", kT=1e-4, max_bodies=1, max_beads=1)
    reps = lbrb.make_replicas([((1, 1, 1), 5), ((2, 3, 1), 6)])
    sim = lbrb.Simulation(p, reps)
    sim.set_mask(1, np.ones(6, dtype=np.uint8))   # all boundary: no fluid node at all
    sim.step(10)
    t0, _, f0, rc0 = sim.observables(0, fields=True)
    t1, _, f1, rc1 = sim.observables(1, fields=True)
    assert rc0 == 0 and rc1 == 0
    assert abs(t0["mass"] - 1.0) < 1e-14
    assert t1["mass"] == 0.0 and np.all(f1 == 0.0)
    assert sim.node_counts(1) == (6, 0)
    from oracle import pyoracle as po
    o = po.OracleSim((1, 1, 1), po.make_params(kT=1e-4, seed=5))
    o.step(10)
    assert np.abs(sim.populations(0).reshape(19) - o.populations().reshape(19)).max() < 1e-15


def test_error_codes():
    p = lbrb.make_params("f32", max_bodies=1, max_beads=4)
    reps = lbrb.make_replicas([((8, 8, 8), 1)])
    sim = lbrb.Simulation(p, reps)
    # rows with two fluid runs are accepted; the wall between them is no fluid node
    m = np.zeros((8, 8, 8), dtype=np.uint8)
    m[:, :, 3] = 1
    sim.set_mask(0, m)
    assert sim.node_counts(0) == (512, 448)
    with pytest.raises(lbrb.LBError) as e:
        sim.add_body(0, np.zeros((5, 3)), 1.0, (1, 1, 1), (4, 4, 4))
    assert e.value.code == lbrb.LB_ERR_CAPACITY
    with pytest.raises(lbrb.LBError) as e:
        sim.add_body(0, np.zeros((1, 3)), -1.0, (1, 1, 1), (4, 4, 4))
    assert e.value.code == lbrb.LB_ERR_ARG
    with pytest.raises(lbrb.LBError) as e:
        sim.add_body(3, np.zeros((1, 3)), 1.0, (1, 1, 1), (4, 4, 4))
    assert e.value.code == lbrb.LB_ERR_ARG
    sim.step(1)
    with pytest.raises(lbrb.LBError) as e:
        sim.set_mask(0, np.zeros((8, 8, 8), dtype=np.uint8))
    assert e.value.code == lbrb.LB_ERR_STATE
    with pytest.raises(lbrb.LBError):
        sim.set_graph_steps(3)
    bad = lbrb.make_params("f32", tau_shear=0.5)
    assert lbrb.lb_workspace_bytes(bad, reps) == 0


def test_unstable_run_is_reported():
    """gamma as specified (20) diverges; the library reports it instead of failing silently."""
    wl = W.workload(1, gamma=W.GAMMA_AS_SPECIFIED)
    wl["precision"] = "f32"
    sim = gpu_from_workload(wl)
    sim.step(60)
    t, _, _, rc = sim.observables(0, check=False)
    assert rc == lbrb.LB_ERR_UNSTABLE


@pytest.mark.parametrize("shape", [(1, 1, 24), (24, 1, 1), (1, 16, 1), (3, 2, 1)])
@pytest.mark.parametrize("precision", ["f64", "f32"])
def test_degenerate_boxes_with_a_body(shape, precision):
    """Boxes one node thick: periodic neighbours are the node itself, and the 8 stencil corners
    of a bead fall onto the same few nodes (several lanes of one bead spread to one node)."""
    rng = np.random.default_rng(sum(shape))
    offs = np.vstack([np.zeros(3), rng.normal(0, 0.8, (6, 3))])
    m, I = 5.0, (2.0, 2.0, 2.0)
    centre = np.array(shape, float) / 2 + 0.13
    wl = dict(name="degenerate", precision=precision, steps=10,
              params=W.default_params(kT=4e-5, g_ext=(1e-5, -2e-6, 3e-6)),
              replicas=[dict(shape=shape, seed=31, mask=None,
                             bodies=[W.body_record(offs, m, I, centre,
                                                   quat=W.random_quaternion(rng),
                                                   vel=(1e-3, 0, -1e-3), gamma=W.GAMMA_FREE)])])
    gpu = gpu_from_workload(wl)
    gpu.set_graph_steps(0)
    orc = oracle_from_workload(wl)
    gpu.step(10)
    orc.step(10)
    e = compare(gpu, orc)
    print(shape, precision, {k: f"{v:.3g}" for k, v in e.items() if isinstance(v, float)})
    tol_u, tol_r = (1e-11, 1e-13) if precision == "f64" else (1e-5, 1e-6)
    assert e["rc"] == 0 and e["finite"]
    assert e["rho"] <= tol_r and e["u_abs"] <= tol_u * max(e["u_scale"], 1e-12)
    for k in ("vel", "omega", "force", "torque"):
        assert e["body_" + k] <= tol_u * max(e["scale_" + k], 1e-14) + 1e-15, k
    assert e["body_pos"] <= tol_r * 100 and e["body_quat"] <= tol_r * 100


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_store_policy_does_not_change_results(precision):
    """Non-temporal and ordinary population stores write the same values."""
    wl = W.workload(1)
    wl["params"]["kT"] = 4e-5
    out = []
    for policy in (lbrb.LB_STORES_CACHED, lbrb.LB_STORES_STREAMING, lbrb.LB_STORES_AUTO):
        gpu = gpu_from_workload(wl, precision=precision)
        gpu.set_store_policy(policy)
        gpu.step(30)
        out.append(gpu.populations(0))
        gpu.close()
    assert np.array_equal(out[0], out[1]) and np.array_equal(out[0], out[2])
    with pytest.raises(lbrb.LBError):
        gpu = gpu_from_workload(wl, precision=precision)
        gpu.set_store_policy(7)


def test_saved_state_does_not_depend_on_the_buffer():
    """Every byte of a saved state is written: buffers prefilled differently end up equal."""
    import ctypes
    import torch
    wl = _thermal_sphere("f64")
    sim = gpu_from_workload(wl)
    sim.step(5)
    L = lbrb.library()
    n = ctypes.c_size_t(0)
    assert L.lb_save_state(sim.ctx, None, ctypes.byref(n)) == lbrb.LB_OK
    out = []
    for fill in (0x00, 0xA5):
        buf = torch.full((n.value,), fill, dtype=torch.uint8, device=sim.device)
        assert L.lb_save_state(sim.ctx, ctypes.c_void_p(buf.data_ptr()), ctypes.byref(n)) == lbrb.LB_OK
        out.append(buf.cpu().numpy())
    assert np.array_equal(out[0], out[1])
    sim.close()


@pytest.mark.parametrize("case", ["pore_f32", "pore_f64", "dense_f32"])
def test_injected_nan_is_reported_and_a_checkpoint_restores_the_run_bitwise(case):
    """Failure detection and recovery: a NaN written into one population (lb_inject_nan)
    spreads, lb_observables reports LB_ERR_UNSTABLE, and loading the checkpoint taken before
    it reruns the same steps bit for bit (graph replays and eager steps mixed)."""
    from tests.test_gpu_parity import pore_case
    precision = case[-3:]
    if case.startswith("pore"):
        wl = pore_case(precision, 4e-5)
    else:
        wl = dict(name="dense", precision=precision, steps=10,
                  params=W.default_params(kT=4e-5, g_ext=(1e-6, 0.0, -2e-6)),
                  replicas=[dict(shape=(20, 18, 16), seed=4, mask=None, bodies=[])])
    sim = gpu_from_workload(wl)
    sim.set_graph_steps(4)
    sim.step(6)
    ck = sim.save_state().clone()
    sim.step(11)
    want = sim.save_state().cpu().numpy()
    assert sim.observables(0, check=False)[3] == lbrb.LB_OK
    mask = wl["replicas"][0]["mask"]
    nx, ny, nz = wl["replicas"][0]["shape"]
    x, y, z = nx // 2, ny // 2, nz // 2
    assert mask is None or mask[z, y, x] == 0
    sim.load_state(ck)
    sim.inject_nan(0, x, y, z, 7)
    sim.step(3)
    t, _, _, rc = sim.observables(0, check=False)
    assert rc == lbrb.LB_ERR_UNSTABLE and not t["finite"]
    sim.load_state(ck)
    assert sim.observables(0, check=False)[3] == lbrb.LB_OK
    sim.step(11)
    assert np.array_equal(sim.save_state().cpu().numpy(), want)
    # a boundary node, a node outside the box and a population out of range are refused
    bad = [(nx, 0, 0, 0), (0, 0, 0, 19), (0, 0, -1, 0)]
    if mask is not None:
        zz, yy, xx = np.argwhere(mask != 0)[0]
        bad.append((int(xx), int(yy), int(zz), 1))
    for args in bad:
        with pytest.raises(lbrb.LBError) as e:
            sim.inject_nan(0, *args)
        assert e.value.code == lbrb.LB_ERR_ARG
    sim.close()


@pytest.mark.parametrize("precision", ["f32", "f64"])
def test_observables_write_every_node_and_only_their_replica(precision):
    """A field buffer holding other values: boundary nodes of a pore stored along z, of an obstacle
    between fluid runs and of a box without fluid come back as zeros, and the bodies are the
    replica's, whatever order they were added in."""
    import torch
    block = np.zeros((20, 13, 17), dtype=np.uint8)
    block[5:9, 3:8, 4:9] = 1
    masks = [W.pore_mask(21, 21, 40, 8.0), block, np.ones((6, 5, 7), dtype=np.uint8), None]
    shapes = [m.shape[::-1] if m is not None else (9, 10, 11) for m in masks]
    offs = W.sphere_beads(1.5, 30)
    mass, inertia = W.solid_body_mass_inertia(1.0, 1.5, 1.5, 1.5)
    params = lbrb.make_params(precision=precision, max_bodies=5, max_beads=5 * len(offs), kT=4e-5)
    sim = lbrb.Simulation(params, lbrb.make_replicas([(s, 7 + k) for k, s in enumerate(shapes)]))
    for r, m in enumerate(masks):
        if m is not None:
            sim.set_mask(r, m)
    order = [(1, 0.3), (0, 0.1), (1, 0.2), (3, 0.4), (0, 0.5)]
    for r, v in order:
        sim.add_body(r, offs, mass, inertia, np.array(shapes[r]) / 2.0, vel=(0.001 * v, 0, 0),
                     gamma=W.GAMMA_FREE, fixed=v == 0.4)
    assert sim.row_axis(0) == 2
    sim.step(3)
    for r, m in enumerate(masks):
        n = 4 * int(np.prod(shapes[r]))
        buf = torch.full((n + 8,), 77.0, dtype=sim.dtype, device="cuda:0")
        rc, tot, bodies = lbrb.lb_observables(sim.ctx, r, sim.n_bodies[r], buf.data_ptr(), check=False)
        assert rc == 0
        f = buf.cpu().numpy()
        assert np.all(f[n:] == 77.0)
        f = f[:n].reshape(*shapes[r][::-1], 4)
        solid = np.zeros(f.shape[:3], bool) if m is None else m != 0
        assert np.all(f[solid] == 0.0) and np.all(np.abs(f[~solid][:, 0] - 1.0) < 0.1)
        # the sum over the fluid nodes, to the rounding of the fields
        assert abs(tot.mass - float(f[..., 0].astype(np.float64).sum())) <= 1e-6 * max(1.0, tot.mass)
        mine = [v for q, v in order if q == r]
        assert len(bodies) == len(mine)
        for b, v in zip(bodies, mine):
            assert np.allclose(b.pos[:], np.array(shapes[r]) / 2.0, atol=0.1)
        free = [b for b, v in zip(bodies, mine) if v != 0.4]
        p = mass * np.sum([b.vel[:] for b in free], axis=0) if free else np.zeros(3)
        assert np.allclose(tot.body_momentum[:], p, rtol=1e-12, atol=1e-18)
    sim.close()
