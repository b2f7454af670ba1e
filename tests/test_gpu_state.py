"""Host state in and out (lb_set_state, lb_get_state, lb_set_profile and the
stress calls) against the definition in numpy, bit for bit: an FP64 slot holds
the value itself, an FP32 slot n - a_i - E_i(u) rounded to FP32, u the row mean
of u_x summed from x = 0 on; a value a moving half-way wall reflects is stored
without the wall's term, and a Zou-He top wall completes its row.

Shapes: one node, one row, channels of few rows (staged three rows at a time
in FP32), 64 x 64 and one row more (the largest staged at once, and the first
in several parts), rows longer than a workgroup, a ragged last tile."""
import numpy as np
import pytest

from paper_1310_7450_amd import workloads
from paper_1310_7450_amd.lbnlm import ChannelSpec

pytestmark = pytest.mark.gpu

CX = np.array([0, 1, 0, -1, 0, 1, -1, -1, 1])
CY = np.array([0, 0, 1, 0, -1, 1, 1, -1, -1])
OPP = np.array([0, 3, 4, 1, 2, 7, 8, 5, 6])
W = np.array([4 / 9] + [1 / 9] * 4 + [1 / 36] * 4)
SHAPES = [(1, 1), (5, 1), (1, 70), (3, 2), (1000, 4), (2048, 5), (900, 6), (700, 7), (64, 64), (64, 65), (300, 97),
          (8, 3000)]


def spec(nx, ny, **kw):
    return ChannelSpec(nx=nx, ny=ny, force=3e-6, tau_lb=0.8, G=2e-4, tau0=500.0, gamma_c=0.1, eps=0.01, visc_split=0.3,
                       **kw)


def stored_and_read(c, pops, P, t, fp32):
    """What lb_get_state returns after lb_set_state(pops, P, t)."""
    f = pops.copy()
    if c.top_wall == "zou_he":
        g = f[:, -1].copy()
        s = (g[0] + g[1] + g[3]) + 2.0 * (g[2] + g[5] + g[6])
        d87 = (s * c.wall_velocity - 0.5 * c.force) - ((g[1] - g[3]) + (g[5] - g[6]))
        f[4, -1], f[8, -1], f[7, -1] = g[2], 0.5 * ((g[5] + g[6]) + d87), 0.5 * ((g[5] + g[6]) - d87)
    out, trace = f.copy(), P.copy()
    uw = c.wall_velocity if c.top_wall != "zou_he" and t >= 1 else 0.0
    wall = -6.0 * W[OPP] * CX[OPP] * uw
    ur = np.zeros(c.ny)
    if fp32:
        rho, jx = np.zeros((c.ny, c.nx)), np.zeros((c.ny, c.nx))
        for i in range(9):
            rho = rho + f[i]
            jx = jx + CX[i] * f[i]
        ur = (np.cumsum(jx / rho, axis=1)[:, -1] / c.nx).astype(np.float32).astype(np.float64)
        trace = P.astype(np.float32).astype(np.float64)
    for i in range(9):
        for y in range(c.ny):
            ys = y - CY[i]
            # the stored population and row, and what was taken off it
            p, row, term = (OPP[i], y, wall[i] if ys >= c.ny else 0.0) if not 0 <= ys < c.ny else (i, ys, None)
            v = f[i, y] if term is None else f[i, y] - term
            if fp32:
                e = W[p] * (3.0 * CX[p] * ur[row] + (4.5 * CX[p] * CX[p] - 1.5) * ur[row] * ur[row])
                v = (v - W[p] - e).astype(np.float32).astype(np.float64) + W[p] + e
            out[i, y] = v if term is None else v + term
    if c.top_wall == "zou_he":
        g = out[:, -1].copy()
        s = (g[0] + g[1] + g[3]) + 2.0 * (g[2] + g[5] + g[6])
        d87 = (s * c.wall_velocity - 0.5 * c.force) - ((g[1] - g[3]) + (g[5] - g[6]))
        out[4, -1], out[8, -1], out[7, -1] = g[2], 0.5 * ((g[5] + g[6]) + d87), 0.5 * ((g[5] + g[6]) - d87)
    return out, trace


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("wall", ["rest", "moving", "zou_he"])
@pytest.mark.parametrize("shape", SHAPES)
def test_state_in_and_out(shape, wall, precision):
    from paper_1310_7450_amd import Solver
    nx, ny = shape
    kw = {"rest": {}, "moving": {"wall_velocity": 0.03},
          "zou_he": {"wall_velocity": 0.03, "top_wall": "zou_he"}}[wall]
    if wall == "zou_he" and ny < 2:
        return
    # a channel on each side, whose state must stay as it is
    beside = spec(12, 9)
    chans = [beside, spec(nx, ny, t_startup=50, **kw), beside]
    pops, P = workloads.random_state(nx, ny, seed=nx + ny)
    with Solver(chans, precision=precision, obs_every=20) as s:
        s.set_state(1, pops, P, 7)
        rest = s.get_state(0)
        want = stored_and_read(chans[1], pops, P, 7, precision == "fp32")
        for _ in range(2):  # reading changes nothing
            got = s.get_state(1)
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1], want[1])
        assert s.observe(1, "step") == 7
        for ch in (0, 2):
            side = s.get_state(ch)
            assert np.array_equal(side[0], rest[0]) and np.array_equal(side[1], rest[1])
        # a state read between two steps leaves the run as it is
        s.step(3)
        s.get_state(1)
        s.step(2)
        a = s.get_state(1)
        s.set_state(1, pops, P, 7)
        s.step(5)
        b = s.get_state(1)
        if precision == "fp64":
            assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", SHAPES)
def test_profile_is_that_state(shape, precision):
    """lb_set_profile equals lb_set_state of the equilibrium it documents."""
    from paper_1310_7450_amd import Solver
    nx, ny = shape
    rng = np.random.default_rng(nx * ny)
    u, n1 = 0.05 * rng.standard_normal(ny), 1e-3 * rng.standard_normal(ny)
    rho = 1.0 - 1.5 * n1
    pops = np.empty((9, ny, nx))
    for i in range(9):
        cu = CX[i] * u
        pops[i] = (W[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * (u * u)))[:, None]
    with Solver([spec(nx, ny)], precision=precision) as s:
        s.set_profile(0, u, n1)
        a = s.get_state(0)
        s.set_state(0, pops, np.repeat(n1[:, None], nx, axis=1), 0)
        b = s.get_state(0)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(1, 1), (64, 65), (2048, 5)])
def test_stress_in_and_out(shape, precision):
    from paper_1310_7450_amd import Solver
    nx, ny = shape
    chans = [spec(12, 9), spec(nx, ny), spec(12, 9)]
    sigma = workloads.random_stress(nx, ny, seed=5)
    with Solver(chans, precision=precision, viscoelastic=True) as s:
        before = s.get_state(1)
        s.set_stress(1, sigma)
        want = sigma if precision == "fp64" else sigma.astype(np.float32).astype(np.float64)
        assert np.array_equal(s.get_stress(1), want) and np.array_equal(s.get_stress(1), want)
        assert not s.get_stress(0).any() and not s.get_stress(2).any()
        after = s.get_state(1)
        assert np.array_equal(after[0], before[0]) and np.array_equal(after[1], before[1])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("shape", [(64, 64), (241, 17), (128, 256), (331, 99)])
def test_stress_calls_leave_a_run_alone(shape, precision):
    """Stress in and out on both sides of the sizes up to which it has staging
    of its own (4096 nodes) and is read through the host (32,768), also
    between steps, after which either buffer may be current."""
    from paper_1310_7450_amd import Solver
    nx, ny = shape
    chans = [spec(12, 9), spec(nx, ny), spec(12, 9)]
    pops, P = workloads.random_state(nx, ny, seed=nx)
    sigma = workloads.random_stress(nx, ny, seed=ny)
    runs = []
    for look in (True, False):
        with Solver(chans, precision=precision, obs_every=20, viscoelastic=True, steps_per_sweep=1) as s:
            for n in (3, 1, 2):
                s.set_state(1, pops, P, 7)
                s.set_stress(1, sigma)
                if look:
                    want = sigma if precision == "fp64" else sigma.astype(np.float32).astype(np.float64)
                    assert np.array_equal(s.get_stress(1), want)
                s.step(n)
                if look:
                    assert np.array_equal(s.get_stress(1), s.get_stress(1))
                    s.get_state(1)
                s.step(2)
            runs.append([a for ch in range(3) for a in (*s.get_state(ch), s.get_stress(ch))])
    assert all(np.array_equal(a, b) for a, b in zip(*runs))
