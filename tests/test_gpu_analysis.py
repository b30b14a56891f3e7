"""Trajectory analysis on the GPU against the oracle (oracle/analysis.py).

- seeded synthetic trajectories (random walks of centres around a pore axis, random small
  rotations): the lab-, body- and pore-frame series, the radial coordinate, the MSDs of every
  series, the lab rotational MSD and the radially binned MSD, element by element;
- a long trajectory (200,000 frames) for the chunked sums;
- edge cases: one frame, the largest lag, one body;
- a trajectory recorded from a thermal GPU simulation: the same comparisons, and the lag-1
  identity of the body and lab frames (a rotation keeps lengths).
Tolerances: the GPU sums each body's increments in 256 chunks and the oracle in one sequence,
so the cumulative series agree to rounding of the running sum (1e-12 of its magnitude); MSDs
to 1e-10 relative; the rotational MSD to 1e-8 relative (arccos near 1 amplifies the rounding
of the dot product); bin counts exactly.
"""
import numpy as np
import pytest

from oracle import analysis as OA
from paper_1604_01829_amd import analysis as GA
from paper_1604_01829_amd import lbrb
from paper_1604_01829_amd import workloads as W

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def _host(t):
    return t.cpu().numpy()


def _close(g, o, rel, what):
    scale = max(1.0, float(np.abs(o).max()))
    err = float(np.abs(g - o).max())
    print(f"{what}: max err {err:.3g} (scale {scale:.3g})", flush=True)
    assert err <= rel * scale, what


def _compare_all(traj, centre, n_lags, edges, ref):
    t = _dev(traj)
    # series (oracle frame-major, GPU body-major)
    lab_o = OA.lab_frame(traj).transpose(1, 0, 2)
    body_o = np.concatenate([OA.body_frame_translation(traj), OA.body_frame_rotation(traj)],
                            axis=2).transpose(1, 0, 2)
    pore_o, rad_o = OA.pore_frame(traj, centre)
    pore_o = pore_o.transpose(1, 0, 2)
    lab_g, body_g = GA.lab_frame(t), GA.body_frame(t)
    pore_g, rad_g = GA.pore_frame(t, centre)
    _close(_host(lab_g), lab_o, 1e-12, "lab frame")
    _close(_host(body_g), body_o, 1e-12, "body frame")
    _close(_host(pore_g), pore_o, 1e-12, "pore frame")
    _close(_host(rad_g), rad_o.T, 1e-14, "radial")
    for name, g, o in (("lab", lab_g, lab_o), ("body", body_g, body_o), ("pore", pore_g, pore_o)):
        mg = _host(GA.msd(g, n_lags))
        mo = OA.msd(o.transpose(1, 0, 2), n_lags)
        _close(mg / np.abs(mo).max(), mo / np.abs(mo).max(), 1e-10, f"msd {name}")
    rg = _host(GA.rotation_msd(t, ref, n_lags))
    ro = OA.rotation_msd(traj, ref, n_lags)
    assert np.abs(rg - ro).max() <= 1e-8 * np.abs(ro).max(), "rotation msd"
    sg, cg = GA.binned_msd(pore_g, rad_g, edges, n_lags)
    so, co = OA.binned_msd(pore_o.transpose(1, 0, 2), rad_o, edges, n_lags)
    assert np.array_equal(_host(cg), co), "bin counts"
    _close(_host(sg) / max(1.0, np.abs(so).max()), so / max(1.0, np.abs(so).max()), 1e-10,
           "binned msd")
    return lab_g, body_g


@pytest.mark.parametrize("n_frames,n_bodies", [(3000, 4), (257, 1), (1000, 3)])
def test_synthetic_trajectories(n_frames, n_bodies):
    centre = (32.0, 30.0)
    traj = W.synthetic_trajectory(n_frames, n_bodies, seed=n_frames + n_bodies, centre=centre)
    ref = np.random.default_rng(7).normal(size=(n_bodies, 3))
    _compare_all(traj, centre, min(60, n_frames - 1), [0.0, 3.0, 5.0, 7.0, 100.0], ref)


@pytest.mark.parametrize("n_frames,n_bodies,n_lags", [(1000, 2, 150), (300, 1, 299)])
def test_lags_over_several_blocks(n_frames, n_bodies, n_lags):
    """More lags than one workgroup's block of 64 (and not a multiple of it), up to the
    largest, n_frames - 1."""
    centre = (32.0, 30.0)
    traj = W.synthetic_trajectory(n_frames, n_bodies, seed=5 + n_lags, centre=centre)
    ref = np.random.default_rng(8).normal(size=(n_bodies, 3))
    _compare_all(traj, centre, n_lags, [0.0, 4.0, 100.0], ref)


@pytest.mark.parametrize("edges", [np.linspace(2.0, 9.0, 9),          # 8 bins, the tiled kernel
                                   np.linspace(0.0, 12.0, 13)],       # 12 bins, one workgroup per bin
                         ids=["8_bins", "12_bins"])
def test_binned_msd_bin_counts(edges):
    """Binned MSD with the most bins the tiled kernel takes and with more (the per-bin
    kernel); origins outside every bin (radius below 2) are left out."""
    centre = (32.0, 30.0)
    traj = W.synthetic_trajectory(1500, 3, seed=44, centre=centre)
    t = _dev(traj)
    pore_o, rad_o = OA.pore_frame(traj, centre)
    pore_g, rad_g = GA.pore_frame(t, centre)
    sg, cg = GA.binned_msd(pore_g, rad_g, list(edges), 100)
    so, co = OA.binned_msd(pore_o, rad_o, list(edges), 100)
    assert np.array_equal(_host(cg), co), "bin counts"
    scale = max(1.0, np.abs(so).max())
    _close(_host(sg) / scale, so / scale, 1e-10, "binned msd")


def test_long_trajectory():
    traj = W.synthetic_trajectory(200000, 1, seed=99, step=0.02, rot_step=0.02,
                                  centre=(64.0, 64.0), radius=(10.0, 20.0))
    t = _dev(traj)
    g = _host(GA.body_frame(t))[0]
    o = np.concatenate([OA.body_frame_translation(traj), OA.body_frame_rotation(traj)], axis=2)[:, 0]
    _close(g, o, 1e-12, "body frame, 200000 frames")
    mg = _host(GA.msd(GA.body_frame(t), 25))[0]
    mo = OA.msd(o[:, None, :], 25)[0]
    _close(mg / np.abs(mo).max(), mo / np.abs(mo).max(), 1e-10, "msd, 200000 frames")


def test_edge_cases():
    import torch
    traj = W.synthetic_trajectory(1, 2, seed=3)
    assert np.array_equal(_host(GA.body_frame(_dev(traj))), np.zeros((2, 1, 6)))
    traj = W.synthetic_trajectory(12, 1, seed=4)
    t = _dev(traj)
    m = _host(GA.msd(GA.lab_frame(t), 11))
    mo = OA.msd(OA.lab_frame(traj), 11)
    assert np.abs(m - mo).max() <= 1e-12 * np.abs(mo).max()
    L = lbrb.library()
    out = torch.empty(64, dtype=torch.float64, device="cuda:0")
    s = torch.cuda.current_stream().cuda_stream
    assert L.lb_traj_msd(t.data_ptr(), 12, 1, 3, 12, out.data_ptr(), s) == lbrb.LB_ERR_ARG
    assert L.lb_traj_msd(t.data_ptr(), 12, 1, 7, 3, out.data_ptr(), s) == lbrb.LB_ERR_ARG
    assert L.lb_traj_binned_msd(t.data_ptr(), t.data_ptr(), 12, 1, 4, t.data_ptr(), 1, 3,
                                  out.data_ptr(), out.data_ptr(), s) == lbrb.LB_ERR_ARG


def test_recorded_simulation_trajectory():
    R = 3.0
    offs = W.sphere_beads(R, 250)
    m, I = W.solid_body_mass_inertia(1.0, R, R, R)
    wl = dict(name="rec", precision="f32", steps=0, params=W.default_params(kT=4e-5),
              replicas=[dict(shape=(24, 24, 24), seed=11, mask=None,
                             bodies=[W.body_record(offs, m, I, (12.3, 11.6, 12.1),
                                                   gamma=W.GAMMA_FREE),
                                     W.body_record(W.ellipsoid_beads(4.0, 2.0, 2.0),
                                                   *W.solid_body_mass_inertia(1.0, 4, 2, 2),
                                                   (4.0, 5.0, 3.0), quat=(0.6, 0.2, -0.7, 0.3),
                                                   gamma=W.GAMMA_FREE)])])
    sim = lbrb.simulation_from_workload(wl)
    traj_t = GA.record(sim, 400, 5)
    traj = _host(traj_t)
    assert np.all(np.isfinite(traj))
    ref = np.array([offs[1], [4.0, 0.0, 0.0]])
    lab_g, body_g = _compare_all(traj, (12.0, 12.0), 40, [0.0, 4.0, 8.0, 30.0], ref)
    lab1 = _host(GA.msd(lab_g, 1))[:, 0, :].sum(axis=1)
    body1 = _host(GA.msd(body_g[:, :, :3].contiguous(), 1))[:, 0, :].sum(axis=1)
    assert np.abs(lab1 - body1).max() <= 1e-12 * lab1.max()


@pytest.mark.parametrize("n_frames,n_bodies,n_lags",
                         [(2, 3, 1), (512, 2, 130), (513, 1, 512), (514, 2, 17), (1026, 1, 1025),
                          (300, 260, 20)])
def test_tile_and_segment_edges(n_frames, n_bodies, n_lags):
    """Frames around the 512 intervals of a segment of the series, lags around the 16 and 128 of
    a workgroup, the last lag, and bodies enough for the wide lag blocks."""
    centre = (32.0, 30.0)
    traj = W.synthetic_trajectory(n_frames, n_bodies, seed=n_frames + n_lags, centre=centre,
                                  rot_step=0.2)
    ref = np.random.default_rng(9).normal(size=(n_bodies, 3))
    _compare_all(traj, centre, n_lags, [0.0, 3.0, 5.0, 100.0], ref)


@pytest.mark.parametrize("n_lags", [60, 300])     # one lag per lane, four
def test_binned_msd_bin_of_every_frame_its_own(n_lags):
    """Bins that change with every origin (and origins outside all of them)."""
    rng = np.random.default_rng(12)
    F, B = 1300, 2
    series = np.cumsum(rng.normal(size=(F, B, 3)), axis=0)
    radial = rng.uniform(0.0, 10.0, size=(F, B))
    edges = [0.5, 2.0, 3.0, 5.0, 6.0, 8.0, 9.0]
    sg, cg = GA.binned_msd(_dev(series.transpose(1, 0, 2)), _dev(radial.T), edges, n_lags)
    so, co = OA.binned_msd(series, radial, edges, n_lags)
    assert np.array_equal(_host(cg), co), "bin counts"
    _close(_host(sg) / np.abs(so).max(), so / np.abs(so).max(), 1e-10, "binned msd")


def test_non_finite_pose_reaches_the_lags_that_use_it():
    traj = W.synthetic_trajectory(700, 2, seed=21)
    traj[400, 1, 3:] = np.nan
    ref = np.array([[1.0, 0.0, 0.0], [0.0, 1.0, 0.5]])
    g = _host(GA.rotation_msd(_dev(traj), ref, 450))
    o = OA.rotation_msd(traj, ref, 450)
    assert np.array_equal(np.isnan(g), np.isnan(o))
    assert np.abs(g - o)[~np.isnan(o)].max() <= 1e-8 * np.nanmax(o)


@pytest.mark.parametrize("lo,hi", [(60.0, 90.0), (90.0, 150.0), (150.0, 180.0)])
def test_wide_angles_are_as_accurate_as_the_arccosine(lo, hi):
    """Poses at rest but for one frame, turned by the angle: of the 4096 terms of lag 1 two are not
    zero, and equal, so the mean is exact and shows the error of one term.  Its r.m.s. over 2000
    angles is at most 1.1 times that of the arccosine of the FP64 cosine (the r.m.s. of 2000 values
    scatters by 2 %), both from long double."""
    import torch
    B, F = 2000, 4097
    th = np.radians(np.random.default_rng(3).uniform(lo, hi, B))
    w, z = np.cos(th / 2), np.sin(th / 2)
    traj = torch.zeros((F, B, 7), dtype=torch.float64, device="cuda:0")
    traj[:, :, 3] = 1.0
    traj[1000, :, 3] = _dev(w)
    traj[1000, :, 6] = _dev(z)
    got = 2048.0 * _host(GA.rotation_msd(traj, np.tile([1.0, 0.0, 0.0], (B, 1)), 1))[:, 0]
    wl, zl = w.astype(np.longdouble), z.astype(np.longdouble)
    want = np.arctan2(2 * wl * zl, 1 - 2 * zl * zl) ** 2
    px, py = 1.0 - 2.0 * (z * z), 2.0 * (z * w)
    c = px / np.sqrt(px * px + py * py)
    rms = [float(np.sqrt(np.mean((((v - want) / want) ** 2).astype(np.float64))))
           for v in (got, np.arccos(c) ** 2)]
    print(f"{lo}-{hi} degrees: r.m.s. error {rms[0]:.3g}, the arccosine's {rms[1]:.3g}", flush=True)
    assert rms[0] <= 1.1 * rms[1]


@pytest.mark.parametrize("n_frames,n_bodies,n_lags",
                         [(1, 1, 0), (2, 1, 1), (257, 2, 65), (1536, 1, 17), (1537, 1, 1536), (4112, 1, 15),
                          (1300, 40, 129), (700, 90, 257), (531, 40, 530)])
def test_msd_short_narrow_and_wide(n_frames, n_bodies, n_lags):
    """Every kernel of the MSD (by the estimates: the short one up to a few hundred frames, for one
    component longer; 16 lags a workgroup for few bodies and lags; 128), at the ends of their blocks
    and of the trajectory, for 1 to 6 components, against the oracle: both FP64 sums of up to 4112
    terms in different orders, 1e-12 of the largest."""
    rng = np.random.default_rng(n_frames + n_lags)
    s = np.cumsum(rng.normal(size=(n_frames, n_bodies, 6)), axis=0)
    for k in (1, 2, 3, 6):
        if n_lags == 0:
            with pytest.raises(lbrb.LBError):
                GA.msd(_dev(s[:, :, :k].transpose(1, 0, 2)), 1)
            continue
        g = _host(GA.msd(_dev(s[:, :, :k].transpose(1, 0, 2)), n_lags))
        o = OA.msd(s[:, :, :k], n_lags)
        assert g.shape == o.shape
        assert np.abs(g - o).max() <= 1e-12 * np.abs(o).max()


@pytest.mark.parametrize("what,n_frames,n_bodies,n_lags,us",
                         [("msd", 20, 20000, 10, 600), ("msd", 1000, 48, 300, 150),
                          ("rotation", 20, 20000, 10, 300), ("binned", 256, 8, 255, 27)])
def test_short_trajectories_take_no_tiles(what, n_frames, n_bodies, n_lags, us):
    """Many bodies recorded a few times: blocks as long as a long trajectory's would be idle (2727,
    237, 681 and 34 us for these; 60, 27, 96 and 22 us one lag per lane)."""
    import torch
    if what == "msd":
        s = torch.randn(n_bodies, n_frames, 6 if n_frames == 20 else 3, dtype=torch.float64,
                        device="cuda:0")
        run = lambda: GA.msd(s, n_lags)
    elif what == "binned":
        s = torch.randn(n_bodies, n_frames, 3, dtype=torch.float64, device="cuda:0")
        rad = torch.rand(n_bodies, n_frames, dtype=torch.float64, device="cuda:0")
        e = torch.linspace(0.0, 1.0, 5, dtype=torch.float64, device="cuda:0")
        sums = torch.empty(4 * n_lags * 3, dtype=torch.float64, device="cuda:0")
        counts = torch.empty(4 * n_lags, dtype=torch.float64, device="cuda:0")
        L, stream = lbrb.library(), torch.cuda.current_stream().cuda_stream
        run = lambda: L.lb_traj_binned_msd(s.data_ptr(), rad.data_ptr(), n_frames, n_bodies, 3,
                                           e.data_ptr(), 4, n_lags, sums.data_ptr(),
                                           counts.data_ptr(), stream)
    else:
        t = _dev(W.synthetic_trajectory(n_frames, n_bodies, seed=2))
        ref = np.tile([1.0, 0.0, 0.0], (n_bodies, 1))
        L, out = lbrb.library(), torch.empty(n_bodies * n_lags, dtype=torch.float64, device="cuda:0")
        r = _dev(ref)
        stream = torch.cuda.current_stream().cuda_stream
        run = lambda: L.lb_traj_rotation_msd(t.data_ptr(), n_frames, n_bodies, r.data_ptr(), n_lags,
                                             out.data_ptr(), stream)
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = 1e9
    for _ in range(4):
        run()
        a.record()
        for _ in range(5):
            run()
        b.record()
        b.synchronize()
        best = min(best, 1e3 * a.elapsed_time(b) / 5)
    print(f"{what} {n_bodies} x {n_frames}, {n_lags} lags: {best:.1f} us", flush=True)
    assert best <= us


@pytest.mark.parametrize("n_frames,n_bodies,n_lags",
                         [(2, 1, 1), (65, 2, 64), (300, 1, 65), (1041, 1, 17), (1040, 3, 1039),
                          (900, 120, 129), (257, 90, 256)])
def test_rotation_short_narrow_and_wide(n_frames, n_bodies, n_lags):
    """Every kernel of the rotational MSD at the ends of its blocks and of the trajectory, turning by
    up to half a turn within it, against the oracle (1e-8, as above)."""
    traj = W.synthetic_trajectory(n_frames, n_bodies, seed=n_frames + n_lags, rot_step=0.2)
    ref = np.random.default_rng(n_lags).normal(size=(n_bodies, 3))
    g, o = _host(GA.rotation_msd(_dev(traj), ref, n_lags)), OA.rotation_msd(traj, ref, n_lags)
    _close(g, o, 1e-8, "rotation msd")


@pytest.mark.parametrize("n_bodies", [1, 2])
@pytest.mark.parametrize("n_frames,n_lags", [(5000, 300), (2100, 64), (130, 129)])
def test_binned_msd_of_two_bodies_repeats_bit_for_bit(n_bodies, n_frames, n_lags):
    """One or two bodies: the same bits on every call, for bins that change with every origin, and
    the oracle's sums (up to 5000 terms in another order: 1e-12 of the largest)."""
    rng = np.random.default_rng(n_frames + n_bodies)
    series = np.cumsum(rng.normal(size=(n_frames, n_bodies, 3)), axis=0)
    radial = rng.uniform(0.0, 10.0, size=(n_frames, n_bodies))
    edges = [0.0, 1.0, 2.0, 3.5, 5.0, 6.0, 8.0, 9.0, 9.5]
    s, r = _dev(series.transpose(1, 0, 2)), _dev(radial.T)
    first, counts = (_host(x) for x in GA.binned_msd(s, r, edges, n_lags))
    for _ in range(20):
        again, c = GA.binned_msd(s, r, edges, n_lags)
        np.testing.assert_array_equal(_host(again), first)
        np.testing.assert_array_equal(_host(c), counts)
    so, co = OA.binned_msd(series, radial, edges, n_lags)
    np.testing.assert_array_equal(counts, co)
    assert np.abs(first - so).max() <= 1e-12 * np.abs(so).max()


@pytest.mark.parametrize("n_bodies,k,n_bins", [(1, 1, 8), (2, 2, 3), (3, 1, 1), (3, 2, 8), (5, 3, 2)])
@pytest.mark.parametrize("n_frames,n_lags", [(2, 1), (65, 64), (66, 65), (513, 128), (512, 129), (1025, 511),
                                             (2049, 1), (1300, 1299)])
def test_binned_msd_edges(n_frames, n_lags, n_bodies, k, n_bins):
    """Frames around a wave's 64 origins and the 512 or 1024 of a chunk, lags around a workgroup's 64
    and 256, origins that no, some and every lag reaches; a non-finite frame reaches the sums of
    its own origins and lags only."""
    rng = np.random.default_rng(n_frames + n_lags + n_bodies)
    series = np.cumsum(rng.normal(size=(n_frames, n_bodies, k)), axis=0)
    radial = 5.0 + np.cumsum(rng.normal(size=(n_frames, n_bodies)), axis=0) / 10.0
    edges = np.linspace(3.0, 7.0, n_bins + 1)
    if n_frames > 600:
        series[-40, 0, 0] = np.nan
    g, c = (_host(x) for x in GA.binned_msd(_dev(series.transpose(1, 0, 2)), _dev(radial.T), edges,
                                            n_lags))
    so, co = OA.binned_msd(series, radial, edges, n_lags)
    np.testing.assert_array_equal(c, co)
    np.testing.assert_array_equal(np.isnan(g), np.isnan(so))
    ok = ~np.isnan(so)
    assert np.abs(g - so)[ok].max(initial=0.0) <= 1e-12 * np.abs(so[ok]).max(initial=1.0)
