"""GPU RK4 flow maps (ftle_advect_rk4) against the FP64 oracle, and the
sliding-window pipeline: one advection call over several meshes' windows
feeding one batched FTLE call.

Tolerance: both sides step the same RK4 in float64; they differ only in the
rounding of the velocity's sines and cosines (the GPU forms sin(pi f) as
sinpi(f)), which the flow's stretching amplifies by at most exp(lambda T)
(lambda < 1 on these flows): 1e-9 absolute over T = 15 is ample.  Float32
output adds its own rounding.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2408_02758_amd as F
from workloads import flows, meshes

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("flow,dim", [("double_gyre", 2), ("abc", 3)])
def test_advect_vs_oracle(flow, dim):
    if dim == 2:
        x, _ = meshes.jittered_tri_grid(64, 48, seed=4)
        t0, T, dt = 0.5, 15.0, 0.01
    else:
        x, _ = meshes.kuhn_tet_grid(14)
        t0, T, dt = 0.0, 10.0, 0.02
    ref = oracle.advect_rk4(flow, x, t0, T, dt)
    x64 = torch.as_tensor(x, dtype=torch.float64, device=DEV)
    got = F.advect_rk4(flow, x64, t0, T, dt).cpu().numpy()
    err = np.abs(got - ref).max()
    print(f"[advect {flow} f64] max |d| = {err:.3e}", flush=True)
    assert err < 1e-9
    got32 = F.advect_rk4(flow, x64.float().contiguous(), t0, T, dt).cpu().numpy().astype(np.float64)
    ref32 = oracle.advect_rk4(flow, x.astype(np.float32).astype(np.float64), t0, T, dt)
    assert np.all(np.abs(got32 - ref32) <= 1e-9 + 2 ** -23 * np.abs(ref32))
    # backward in time returns the start up to the RK4 truncation error, which
    # the flow's stretching amplifies (1.3e-6 for the ABC flow at dt = 0.02 over
    # T = 10 and back); and T = 0 is the identity
    back = F.advect_rk4(flow, torch.as_tensor(ref, device=DEV), t0 + T, -T, dt).cpu().numpy()
    assert np.abs(back - x).max() < 1e-5
    assert torch.equal(F.advect_rk4(flow, x64, 1.0, 0.0, dt), x64)


def test_windows_pipeline_vs_oracle():
    """Three meshes, each with its own window (t0, T), advected in one call with
    per-particle times, then their FTLE in one batched call; against the
    oracle's flow maps and FTLE."""
    sides, t0s, Ts = (30, 41, 25), (0.0, 2.5, 7.0), (15.0, 10.0, -12.0)
    geo = [meshes.jittered_tri_grid(s, s, seed=100 + k) for k, s in enumerate(sides)]
    counts = [g[0].shape[0] for g in geo]
    allx = np.concatenate([g[0] for g in geo])
    t0p = np.repeat(t0s, counts)
    Tp = np.repeat(Ts, counts)
    xd = torch.as_tensor(allx, dtype=torch.float64, device=DEV)
    phi = F.advect_rk4("double_gyre", xd, torch.as_tensor(t0p, device=DEV), torch.as_tensor(Tp, device=DEV), 0.01)
    ref_phi = oracle.advect_rk4("double_gyre", allx, t0p, Tp, 0.01)
    assert np.abs(phi.cpu().numpy() - ref_phi).max() < 1e-9
    # the same as one call per window, bit for bit
    off = np.concatenate([[0], np.cumsum(counts)])
    for k in range(3):
        one = F.advect_rk4("double_gyre", xd[off[k]:off[k + 1]].contiguous(), t0s[k], Ts[k], 0.01)
        assert torch.equal(one, phi[off[k]:off[k + 1]])
    ms = [F.Mesh(g[0], g[1], "f64") for g in geo]
    flows_k = [phi[off[k]:off[k + 1]].contiguous() for k in range(3)]
    outs = F.batched(ms, flows_k, list(Ts))
    for k, (g, out) in enumerate(zip(geo, outs)):
        st = oracle.ring1(2, g[0].shape[0], g[1])
        ref = oracle.ftle(2, g[0], ref_phi[off[k]:off[k + 1]], st, Ts[k])
        got = out.cpu().numpy()
        fin = np.isfinite(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        # the flow maps differ by < 1e-9; the stencil differences amplify that by 1/spacing
        assert np.abs(got[fin] - ref[fin]).max() < 1e-6


def test_advect_large_start_time_and_ragged_steps():
    """Double gyre from a start time far from 0 (a large phase omega t) over a
    duration that is not a whole number of steps, forward and backward: the
    kernel's time factor (advanced by rotations, evaluated directly every few
    steps) against the oracle's direct evaluation at every stage."""
    x, _ = meshes.jittered_tri_grid(20, 15, seed=9)
    x64 = torch.as_tensor(x, dtype=torch.float64, device=DEV)
    for t0, T in ((12345.6, 7.305), (-987.25, -3.3333)):
        ref = oracle.advect_rk4("double_gyre", x, t0, T, 0.01)
        got = F.advect_rk4("double_gyre", x64, t0, T, 0.01).cpu().numpy()
        err = np.abs(got - ref).max()
        print(f"[advect double_gyre t0={t0} T={T}] max |d| = {err:.3e}", flush=True)
        assert err < 1e-9


def test_advect_full_2048_sampled():
    """The measured flow map: all 4,194,304 particles of the 2048^2 jittered
    grid (float32 in and out, as the benchmark times it), 3,000 of them
    against the oracle's RK4 on the same float32 starting points."""
    x, _ = meshes.jittered_tri_grid(2048, 2048, seed=7)
    x32 = np.ascontiguousarray(x, dtype=np.float32)
    phi = F.advect_rk4("double_gyre", torch.as_tensor(x32, device=DEV), 0.0, 15.0, 0.01).cpu().numpy()
    sel = np.unique(np.concatenate([np.random.default_rng(2).choice(x32.shape[0], 3000, replace=False),
                                    np.arange(32), np.arange(x32.shape[0] - 32, x32.shape[0])]))
    ref = oracle.advect_rk4("double_gyre", x32[sel].astype(np.float64), 0.0, 15.0, 0.01)
    err = np.abs(phi[sel].astype(np.float64) - ref)
    print(f"[advect 2048^2 sampled] max |d| = {err.max():.3e}", flush=True)
    assert np.all(err <= 1e-9 + 2.0 ** -23 * np.abs(ref))


# ---------------------------------------------------------------------------
# ftle_advect_rk4_grid: a velocity field sampled on a regular grid
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("flow,shift", [("double_gyre", 0.0), ("double_gyre", 2.0 ** 29), ("double_gyre", 2.0 ** 31),
                                        ("abc", 0.0), ("abc", 2.0 ** 29), ("abc", 2.0 ** 31)])
def test_advect_reach(flow, shift):
    """Both step forms, either side of the reach (2^30) that picks between them:
    particles shifted along y (double gyre) or every axis (ABC), mixed with
    unshifted ones and with non-finite ones in the same waves.

    Tolerance: each of the 5 steps rounds the position by at most half its
    spacing u, and the oracle's argument pi y carries at most another u of
    phase; the flow stretches these by less than exp(10 * 0.1) < 3 on the way:
    (5 / 2 + 1) * 3 u < 16 u.  Unshifted particles: 1e-9, as above."""
    x = meshes.jittered_tri_grid(16, 12, seed=9)[0] if flow == "double_gyre" else meshes.kuhn_tet_grid(6)[0]
    n, t0, T, dt = x.shape[0], 0.3, 0.1, 0.02
    far = np.arange(n) % 3 == 0
    x = x.copy()
    if flow == "double_gyre":
        x[far, 1] += shift
    else:
        x[far] += shift
    ref = oracle.advect_rk4(flow, x, t0, T, dt)
    bad = np.arange(n) % 17 == 1
    xb = x.copy()
    xb[bad, 0] = np.where(np.arange(bad.sum()) % 2, np.nan, np.inf)
    got = F.advect_rk4(flow, torch.as_tensor(xb, device=DEV), t0, T, dt).cpu().numpy()
    assert np.isnan(got[bad, 0]).all()
    tol = np.where(far, 16 * np.spacing(max(shift, 1.0)), 1e-9) if shift else np.full(n, 1e-9)
    assert np.all(np.abs(got - ref)[~bad] <= tol[~bad, None])


def test_advect_walls_are_kept():
    """A double-gyre particle on a wall (y an integer, x = 0) stays on it exactly."""
    r = np.random.default_rng(3)
    x = np.stack([r.random(200) * 2, r.integers(-1, 3, 200)], 1).astype(np.float64)
    x[150:, 0], x[150:, 1] = 0.0, r.random(50)
    got = F.advect_rk4("double_gyre", torch.as_tensor(x, device=DEV), 0.2, 15.0, 0.01).cpu().numpy()
    assert np.array_equal(got[:150, 1], x[:150, 1])
    assert np.array_equal(got[150:, 0], x[150:, 0])


@pytest.mark.parametrize("axis", [0, 1])
@pytest.mark.parametrize("dist", [1e-6, 1e-9, 1e-12, 1e-200])
def test_advect_next_to_walls(axis, dist):
    """A double-gyre particle next to the wall x = 0 or y = 0 keeps its distance to
    it to a relative tolerance: the normal velocity is the distance times a
    factor of the other coordinate, in which no absolute error may stand.

    Tolerance: 250 steps round the distance by 2^-53 of it on each side, and
    their velocities (16 roundings, times h v / y <= 0.04) by less; the other
    coordinate's error (at most 2 units of 2^-52 a step on each side, stretched
    by less than exp(5)) moves the factor's integral over T = 5 by less than 15
    of it: 250 * 4 * 2^-52 * 150 * 15 + 250 * 3 * 2^-53 < 6e-10, within 1e-9."""
    r = np.random.default_rng(11)
    x = np.stack([r.random(300) * 2, r.random(300)], 1)
    x[:, axis] = dist * (1 + r.random(300))
    ref = oracle.advect_rk4("double_gyre", x, 0.1, 5.0, 0.02)
    got = F.advect_rk4("double_gyre", torch.as_tensor(x, device=DEV), 0.1, 5.0, 0.02).cpu().numpy()
    err = np.abs(got[:, axis] / ref[:, axis] - 1.0).max()
    print(f"[advect next to a wall, axis {axis}, {dist:g}] max rel |d| = {err:.3e}", flush=True)
    assert err < 1e-9


def test_advect_sines_keep_their_zeros():
    """The ABC flow with A = B = 0 moves a particle at x = z = 0 by T C (cos y, 0, sin y):
    one step shows the sine and cosine of y, which stay relatively exact up to their
    zeros.

    Tolerance: 2 units of 2^-53 for a function, one for each of the five sums and
    products of the step, one for the reference: 8 * 2^-53 = 2^-50 of the value."""
    r = np.random.default_rng(12)
    near = np.arange(1, 20) * np.pi / 2
    y = np.concatenate([r.uniform(-30, 30, 20000), near * (1 + 2.0 ** -30), near * (1 - 2.0 ** -25), -near * (1 + 1e-12),
                        [0.0, np.pi / 2, -np.pi / 2, 1e-300]])
    x = np.zeros((len(y), 3))
    x[:, 1] = y
    got = F.advect_rk4("abc", torch.as_tensor(x, device=DEV), 0.0, 1.0, 1.0, params=(0.0, 0.0, 1.0)).cpu().numpy()
    assert np.array_equal(got[:, 1], y)
    for d, ref in ((0, np.cos(y.astype(np.longdouble))), (2, np.sin(y.astype(np.longdouble)))):
        err = np.abs(got[:, d] - ref)
        print(f"[advect sines, axis {d}] max rel |d| = {np.max(err[ref != 0] / np.abs(ref[ref != 0])):.3e}", flush=True)
        assert np.all(err <= 2.0 ** -50 * np.abs(ref))


@pytest.mark.parametrize("flow", ["double_gyre", "abc"])
def test_advect_reach_by_blocks(flow):
    """The step form is chosen for blocks of 32 steps: particles about the reach, some
    of them on either side of it in different blocks, over two and a half blocks.

    Tolerance, u = 2^-22 the spacing of positions below 2^30: 80 steps round the
    position by u / 2 and carry u of phase, on each side, stretched by less than
    exp(2 * 1.6) < 25: 80 * 3/2 * 2 * 25 u = 6000 u."""
    x = meshes.jittered_tri_grid(25, 20, seed=3)[0] if flow == "double_gyre" else meshes.kuhn_tet_grid(8)[0]
    x = x.copy()
    last = x.shape[1] - 1
    x[:, last] += 2.0 ** 30 - np.random.default_rng(5).uniform(0.0, 20.0, x.shape[0])
    t0, T, dt = 0.3, 1.6, 0.02
    ref = oracle.advect_rk4(flow, x, t0, T, dt)
    got = F.advect_rk4(flow, torch.as_tensor(x, device=DEV), t0, T, dt).cpu().numpy()
    assert np.abs(got - ref).max() <= 6000 * 2.0 ** -22


def _gyre_grid(nx, ny, times):
    """The double gyre at the nodes of an nx x ny grid over [0, 2] x [0, 1]."""
    return flows.sampled_field(flows.double_gyre_velocity, [0.0, 0.0], [2.0 / (nx - 1), 1.0 / (ny - 1)], (nx, ny),
                               times)


def _abc_grid(n):
    """The ABC flow at the nodes of an n^3 grid over [0, 2 pi]^3, and the spacing."""
    h = 2 * np.pi / (n - 1)
    return flows.sampled_field(flows.abc_velocity, [0.0] * 3, [h] * 3, (n, n, n)), h


@pytest.mark.parametrize("vel_dtype", [np.float32, np.float64])
def test_advect_grid_vs_oracle(vel_dtype):
    """Both sides step the same RK4 through the same stored field in float64:
    they differ by rounding only (the summation order of the corner weights),
    amplified by the flow's stretching: 1e-9 over T = 15 as for the analytic flows."""
    times = np.arange(0.0, 20.0 + 1e-9, 0.5)
    vel = _gyre_grid(201, 101, times).astype(vel_dtype)
    x, _ = meshes.jittered_tri_grid(64, 48, seed=5)
    g = np.random.default_rng(2)
    t0s = g.uniform(0.0, 5.0, x.shape[0])
    Ts = g.uniform(-4.0, 15.0, x.shape[0])
    Ts[:7] = 0.0
    ref = oracle.advect_rk4_grid(vel.astype(np.float64), [0.0, 0.0], [0.01, 0.01], 0.0, 0.5, x, t0s, Ts, 0.02)
    vd = torch.as_tensor(vel, device=DEV)
    x64 = torch.as_tensor(x, dtype=torch.float64, device=DEV)
    got = F.advect_rk4_grid(vd, [0.0, 0.0], [0.01, 0.01], 0.0, 0.5, x64, torch.as_tensor(t0s, device=DEV),
                            torch.as_tensor(Ts, device=DEV), 0.02).cpu().numpy()
    err = np.abs(got - ref).max()
    print(f"[advect grid gyre vel={np.dtype(vel_dtype).name}] max |d| = {err:.3e}", flush=True)
    assert err < 1e-9
    assert np.array_equal(got[:7], x[:7])
    # float32 particles: the same up to the output's rounding
    got32 = F.advect_rk4_grid(vd, [0.0, 0.0], [0.01, 0.01], 0.0, 0.5, x64.float().contiguous(), 1.5, 9.0,
                              0.02).cpu().numpy().astype(np.float64)
    ref32 = oracle.advect_rk4_grid(vel.astype(np.float64), [0.0, 0.0], [0.01, 0.01], 0.0, 0.5,
                                   x.astype(np.float32).astype(np.float64), 1.5, 9.0, 0.02)
    assert np.all(np.abs(got32 - ref32) <= 1e-9 + 2 ** -23 * np.abs(ref32))


def test_advect_grid_3d_clamping_and_steady():
    """A sampled ABC field (one slice: steady) in 3D, with particles starting
    outside the grid's box (the nearest box point's velocity), against the oracle."""
    vel, h = _abc_grid(33)
    g = np.random.default_rng(4)
    x = np.concatenate([g.uniform(0.0, 2 * np.pi, size=(3000, 3)), g.uniform(-2.0, 9.0, size=(500, 3))])
    ref = oracle.advect_rk4_grid(vel, [0.0] * 3, [h] * 3, 0.0, 1.0, x, 0.0, 5.0, 0.05)
    got = F.advect_rk4_grid(torch.as_tensor(vel, device=DEV), [0.0] * 3, [h] * 3, 0.0, 1.0,
                            torch.as_tensor(x, device=DEV), 0.0, 5.0, 0.05).cpu().numpy()
    err = np.abs(got - ref).max()
    print(f"[advect grid abc] max |d| = {err:.3e}", flush=True)
    assert err < 1e-9
    assert F.advect_rk4_grid(torch.as_tensor(vel, device=DEV), [0.0] * 3, [h] * 3, 0.0, 1.0,
                             torch.empty(0, 3, dtype=torch.float64, device=DEV), 0.0, 5.0, 0.05).numel() == 0


def test_advect_grid_3d_unsteady():
    """A time-dependent 3D field (the ABC flow with amplitudes varying in
    time) on an anisotropic 17 x 19 x 21 grid at 5 slices, with per-particle
    windows, particles inside and outside the box and times outside the
    slices, float64 and float32 fields, against the oracle."""
    def abc_t(p, t):
        return flows.abc_velocity(p) * (1.0 + 0.3 * torch.sin(0.7 * t))
    shape, spacing, origin = (17, 19, 21), (0.4, 0.35, 0.3), (-0.5, 0.2, -1.0)
    vel = flows.sampled_field(abc_t, origin, spacing, shape, np.arange(5) * 0.8 - 0.4)
    g = np.random.default_rng(6)
    lo, hi = np.array(origin), np.array(origin) + (np.array(shape) - 1) * np.array(spacing)
    x = np.concatenate([g.uniform(lo, hi, size=(2500, 3)), g.uniform(lo - 1.0, hi + 1.0, size=(500, 3))])
    t0s = g.uniform(-1.0, 2.0, x.shape[0])
    Ts = g.uniform(-3.0, 4.0, x.shape[0])
    for vdt in (np.float64, np.float32):
        v = vel.astype(vdt)
        ref = oracle.advect_rk4_grid(v.astype(np.float64), list(origin), list(spacing), -0.4, 0.8, x, t0s, Ts, 0.05)
        got = F.advect_rk4_grid(torch.as_tensor(v, device=DEV), list(origin), list(spacing), -0.4, 0.8,
                                torch.as_tensor(x, device=DEV), torch.as_tensor(t0s, device=DEV),
                                torch.as_tensor(Ts, device=DEV), 0.05).cpu().numpy()
        err = np.abs(got - ref).max()
        print(f"[advect grid 3d unsteady vel={np.dtype(vdt).name}] max |d| = {err:.3e}", flush=True)
        assert err < 1e-9


def test_grid_windows_pipeline_vs_oracle():
    """The sliding-window pipeline from gridded data: three meshes' windows in
    a sampled double gyre (101 x 51 nodes, slices 0.5 apart over [0, 20])
    advected in one call with per-particle times, the same as one call per
    window bit for bit, then one batched FTLE call against the oracle's flow
    maps and FTLE."""
    times = np.arange(41) * 0.5
    vel = torch.as_tensor(_gyre_grid(101, 51, times), device=DEV)
    org, spc = [0.0, 0.0], [0.02, 0.02]
    sides, t0s, Ts = (28, 37, 22), (0.0, 3.25, 19.0), (15.0, 9.5, -11.0)
    geo = [meshes.jittered_tri_grid(s, s, seed=200 + k) for k, s in enumerate(sides)]
    counts = [g[0].shape[0] for g in geo]
    allx = np.concatenate([g[0] for g in geo])
    t0p, Tp = np.repeat(t0s, counts), np.repeat(Ts, counts)
    xd = torch.as_tensor(allx, device=DEV)
    phi = F.advect_rk4_grid(vel, org, spc, 0.0, 0.5, xd, torch.as_tensor(t0p, device=DEV),
                            torch.as_tensor(Tp, device=DEV), 0.01)
    ref_phi = oracle.advect_rk4_grid(vel.cpu().numpy(), org, spc, 0.0, 0.5, allx, t0p, Tp, 0.01)
    assert np.abs(phi.cpu().numpy() - ref_phi).max() < 1e-9
    off = np.concatenate([[0], np.cumsum(counts)])
    for k in range(3):
        one = F.advect_rk4_grid(vel, org, spc, 0.0, 0.5, xd[off[k]:off[k + 1]].contiguous(), t0s[k], Ts[k], 0.01)
        assert torch.equal(one, phi[off[k]:off[k + 1]])
    ms = [F.Mesh(g[0], g[1], "f64") for g in geo]
    outs = F.batched(ms, [phi[off[k]:off[k + 1]].contiguous() for k in range(3)], list(Ts))
    for k, (g, out) in enumerate(zip(geo, outs)):
        st = oracle.ring1(2, g[0].shape[0], g[1])
        ref = oracle.ftle(2, g[0], ref_phi[off[k]:off[k + 1]], st, Ts[k])
        got = out.cpu().numpy()
        fin = np.isfinite(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.abs(got[fin] - ref[fin]).max() < 1e-6


def test_advect_grid_full_2048_sampled():
    """The headline's 2048^2 particles through a double gyre sampled on a
    513 x 257 grid at 61 slices (float32 field, T = 15, dt = 0.01, float32
    output), against the oracle on 20,000 sampled particles."""
    times = np.arange(0.0, 15.0 + 1e-9, 0.25)
    vel = _gyre_grid(513, 257, times).astype(np.float32)
    x, _ = meshes.jittered_tri_grid(2048, 2048, seed=2)
    x32 = torch.as_tensor(x, dtype=torch.float32, device=DEV)
    got = F.advect_rk4_grid(torch.as_tensor(vel, device=DEV), [0.0, 0.0], [2.0 / 512, 1.0 / 256], 0.0, 0.25, x32,
                            0.0, 15.0, 0.01).cpu().numpy().astype(np.float64)
    sel = np.sort(np.random.default_rng(8).choice(x.shape[0], 20000, replace=False))
    ref = oracle.advect_rk4_grid(vel.astype(np.float64), [0.0, 0.0], [2.0 / 512, 1.0 / 256], 0.0, 0.25,
                                 x[sel].astype(np.float32).astype(np.float64), 0.0, 15.0, 0.01)
    err = np.abs(got[sel] - ref) - 2 ** -23 * np.abs(ref)
    print(f"[advect grid 2048^2] max |d| beyond output rounding = {err.max():.3e}", flush=True)
    assert np.all(err <= 1e-9)


@pytest.mark.parametrize("dim,slices,n", [(2, 5, 4096 * 64), (2, 1, 8192 * 64), (3, 3, 2048 * 64), (3, 1, 4096 * 64)])
@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
def test_advect_grid_launch_forms(dim, slices, n, dtype):
    """A particle's path does not depend on the launch: one more than n particles
    take single-wave workgroups, the rest of the calls four-wave ones, with the
    window as numbers or per particle; all bit for bit the same, some particles
    outside the box or not finite."""
    g = torch.Generator(device=DEV).manual_seed(dim * 10 + slices)
    shape = (slices,) + (9, 11, 13)[:dim] + (dim,)
    vel = (torch.rand(shape, generator=g, device=DEV) - 0.5).to(dtype)
    x = torch.rand(n + 1, dim, generator=g, device=DEV, dtype=torch.float64) * 1.4 - 0.2
    x[::1001, 0] = float("nan")
    x[5::1001, 1] = float("inf")
    spacing = [0.125, 0.1, 0.1][:dim]
    args = (vel, [0.0] * dim, spacing, 0.0, 0.3)
    many = F.advect_rk4_grid(*args, x, 0.1, 0.7, 0.09)
    few = x[-1000:].contiguous()
    one = F.advect_rk4_grid(*args, few, 0.1, 0.7, 0.09)
    same = lambda a, b: torch.equal(a.view(torch.int64), b.view(torch.int64))   # noqa: E731 - NaN included
    assert same(many[-1000:].contiguous(), one)
    per = lambda v: torch.full((1000,), v, dtype=torch.float64, device=DEV)   # noqa: E731
    assert same(F.advect_rk4_grid(*args, few, per(0.1), per(0.7), 0.09), one)
    ref = oracle.advect_rk4_grid(vel.double().cpu().numpy(), [0.0] * dim, spacing, 0.0, 0.3, few.cpu().numpy(), 0.1,
                                 0.7, 0.09)
    fin = torch.isfinite(few).all(1).cpu().numpy()
    assert np.abs(one.cpu().numpy()[fin] - ref[fin]).max() < 1e-9


def test_advect_grid_wide_field():
    """A field of 4 GiB and more (64-bit offsets) against a coarse one of the same
    linear velocity (its node values are exact in float32 on both grids): equal
    up to the arithmetic's roundings, 12 steps of at most a few units in the
    last place of positions below 2."""
    m = 16384 + 1
    ax = torch.arange(m, device=DEV, dtype=torch.float32) * 2.0 ** -13
    vel = torch.empty(2, m, m, 2, device=DEV)
    vel[0, :, :, 0], vel[0, :, :, 1] = (ax * 0.25)[:, None], (ax * -0.25)[None, :]
    vel[1] = vel[0] * 2.0
    coarse = vel[:, ::4096, ::4096].contiguous()
    assert vel.numel() * 4 >= 2 ** 32
    x = torch.rand(500, 2, generator=torch.Generator(device=DEV).manual_seed(1), device=DEV, dtype=torch.float64) + 0.5
    fine = F.advect_rk4_grid(vel, [0.0, 0.0], [2.0 ** -13] * 2, 0.0, 2.0, x, 0.0, 1.2, 0.1)
    ref = F.advect_rk4_grid(coarse, [0.0, 0.0], [0.5] * 2, 0.0, 2.0, x, 0.0, 1.2, 0.1)
    assert (fine - ref).abs().max().item() <= 12 * 8 * 2.0 ** -52


def test_wrappers_reject_bad_outputs():
    """The Python wrappers check the output tensor (shape, dtype, device, not
    the input) and the grid's origin and spacing lengths before any launch."""
    x = torch.zeros(10, 2, dtype=torch.float64, device=DEV)
    vel = torch.zeros(2, 3, 4, 2, dtype=torch.float32, device=DEV)
    bad = [torch.empty(9, 2, dtype=torch.float64, device=DEV), torch.empty(10, 2, dtype=torch.float32, device=DEV),
           torch.empty(10, 2, dtype=torch.float64), x]
    for out in bad:
        with pytest.raises(ValueError):
            F.advect_rk4("double_gyre", x, 0.0, 1.0, 0.1, out=out)
        with pytest.raises(ValueError):
            F.advect_rk4_grid(vel, [0.0, 0.0], [1.0, 1.0], 0.0, 1.0, x, 0.0, 1.0, 0.1, out=out)
    with pytest.raises(ValueError):
        F.advect_rk4_grid(vel, [0.0, 0.0, 0.0], [1.0, 1.0], 0.0, 1.0, x, 0.0, 1.0, 0.1)
    ok = F.advect_rk4_grid(vel, [0.0, 0.0], [1.0, 1.0], 0.0, 1.0, x, 0.0, 1.0, 0.1)
    assert torch.equal(ok, x)   # a zero field leaves every particle in place
