"""Many steps per launch on boxes of nodes (small lattices) against one step
per pass, bit for bit: every node update is the same arithmetic, so the box a
node falls in, the steps a launch takes and the halo around it must not show.

Shapes: one node, channels shorter and narrower than a halo, whole channels in
one workgroup and just too large for one (1024 nodes), boxes cut by rows, by
columns and both ways, the periodic wrap of a cut row, ragged last boxes, and
every width class. The two-step kernels of the aligned widths, which larger
lattices keep, are compared with one step per pass at sizes above the boxes'
limits."""
import numpy as np
import pytest

from paper_1310_7450_amd import workloads
from paper_1310_7450_amd.lbnlm import ChannelSpec

pytestmark = pytest.mark.gpu


def spec(nx, ny, **kw):
    base = dict(force=3e-6, tau_lb=0.8, G=2e-4, tau0=500.0, gamma_c=0.1, eps=0.01, visc_split=0.3, t_startup=13)
    base.update(kw)
    return ChannelSpec(nx=nx, ny=ny, **base)


def run(chans, precision, obs_every, steps, steps_per_sweep, viscoelastic=False, stress_force=False):
    """States (and stresses) of every channel after the steps, from seeded
    random states."""
    from paper_1310_7450_amd import Solver
    with Solver(chans, precision=precision, obs_every=obs_every, viscoelastic=viscoelastic,
                stress_force=stress_force, steps_per_sweep=steps_per_sweep) as s:
        for i, c in enumerate(chans):
            s.set_state(i, *workloads.random_state(c.nx, c.ny, seed=31 * c.nx + c.ny + i), 0)
            if viscoelastic:
                s.set_stress(i, workloads.random_stress(c.nx, c.ny, seed=7 + i))
        for n in steps:
            s.step(n)
        out = [s.get_state(i) + ((s.get_stress(i),) if viscoelastic else ()) for i in range(len(chans))]
        assert all(s.observe(i, "step") == sum(steps) for i in range(len(chans)))
    return out


def assert_same(a, b, what):
    for i, (x, y) in enumerate(zip(a, b)):
        for p, q in zip(x, y):
            assert np.isfinite(q).all() and np.array_equal(p, q), (what, i, np.abs(p - q).max())


SHAPES = [(1, 1), (2, 3), (1, 1024), (1, 1025), (8, 128), (8, 129), (16, 7), (64, 16), (64, 90), (33, 31), (65, 2),
          (100, 20), (128, 9), (200, 20), (203, 61), (256, 37), (320, 5), (1000, 30), (1024, 33)]


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("nx,ny", SHAPES)
def test_boxes_equal_one_step(precision, nx, ny):
    """Whole blocks (K = 20: boxes of 1, 2, 5 or 10 steps; the force ends
    inside one) and odd counts of steps off the block boundaries."""
    for steps in ([40], [7, 13, 20, 3]):
        a, b = (run([spec(nx, ny)], precision, 20, steps, sps) for sps in (0, 1))
        assert_same(a, b, (precision, nx, ny, steps))


@pytest.mark.parametrize("obs_every", [2, 6, 14, 100])
def test_boxes_of_every_block_length(obs_every):
    """Block lengths whose half has few divisors, or many."""
    c = [spec(24, 40), spec(8, 50)]
    a, b = (run(c, "fp64", obs_every, [2 * obs_every + 1], sps) for sps in (0, 1))
    assert_same(a, b, obs_every)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("wall", [dict(wall_velocity=1e-3), dict(top_wall="zou_he", wall_velocity=1e-3,
                                                                 nn_pressure=False)])
@pytest.mark.parametrize("viscoelastic", [False, True])
def test_boxes_walls_and_models(precision, wall, viscoelastic):
    """Moving half-way and Zou-He tops (stopping inside a launch), with both
    stress models, in a handle of ragged channels of several widths."""
    c = [spec(8, 64, **wall), spec(200, 20, **wall), spec(1, 9), spec(256, 18, **wall), spec(130, 2, **wall)]
    a, b = (run(c, precision, 20, [40, 9], sps, viscoelastic) for sps in (0, 1))
    assert_same(a, b, (precision, wall, viscoelastic))


def test_boxes_beside_other_channels():
    """A handle that also holds a pressure-driven channel (one step per
    pass inside the same blocks)."""
    c = [spec(8, 40), spec(64, 12, force=0.0, pressure_gradient=1e-6, nn_pressure=False), spec(300, 11)]
    a, b = (run(c, "fp64", 20, [40, 3], sps) for sps in (0, 1))
    assert_same(a, b, "mixed")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("viscoelastic", [False, True])
def test_pressure_many_steps_per_launch(precision, viscoelastic):
    """Boxes of whole columns, whose density every step of a launch takes: one
    and two columns' period, a channel of one box, boxes cut into columns
    (several periods wide with their halo), 64, 65 and more rows of density,
    heights with and without a plan; alone and beside other channels. The
    drive ends inside a launch."""
    kw = dict(force=0.0, pressure_gradient=1e-6, nn_pressure=False, t_startup=31)
    shapes = [(2, 5), (3, 64), (5, 65), (64, 32), (200, 20), (1000, 12), (33, 112), (21, 190), (600, 300), (24, 1)]
    cases = [[spec(nx, ny, **kw)] for nx, ny in shapes]
    cases.append([spec(64, 32, **kw), spec(16, 9, **kw), spec(300, 11), spec(8, 40)])
    for c in cases:
        a, b = (run(c, precision, 40, [80, 7, 1, 4], sps, viscoelastic) for sps in (0, 1))
        assert_same(a, b, (precision, [(q.nx, q.ny) for q in c], viscoelastic))


# the stress as a force: a step reaches three nodes, and the wall's ghost
# stress takes two rows; FP64 round-off over a few steps as below
@pytest.mark.parametrize("wall", [{}, dict(wall_velocity=0.02)])
def test_stress_force_boxes(wall):
    """Boxes of several steps against one step per launch: one node, one and two
    rows, channels of one box, cut by rows, by columns and both ways, ragged;
    alone and in one handle; on both sides of the limit of their kind."""
    kw = dict(nn_pressure=False, t_startup=31, **wall)
    shapes = [(1, 1), (3, 1), (5, 2), (8, 40), (64, 3), (8, 400), (200, 20), (143, 43), (37, 113), (1000, 9)]
    cases = [[spec(nx, ny, **kw)] for nx, ny in shapes] + [[spec(nx, ny, **kw) for nx, ny in shapes[3:8]]]
    cases += [[spec(500, 300, **kw)], [spec(600, 300, **kw)]]
    for c in cases:
        a, b = (run(c, "fp64", 40, [80, 7, 1], sps, stress_force=True) for sps in (0, 1))
        for x, y in zip(a, b):
            for p, q in zip(x, y):
                scale = max(np.abs(q).max(), 1e-300)
                err = np.abs(p - q).max() / scale
                assert err <= 1e-11, ([(s.nx, s.ny) for s in c], err)
        print([(s.nx, s.ny) for s in c], "same" if all(np.array_equal(p, q) for x, y in zip(a, b) for p, q in zip(x, y))
              else "to round-off", flush=True)


# (width, rows) above the boxes' limits; FP32 results of the two-step sweep
# are those of one step per pass, FP64 ones agree to round-off amplified over
# a few steps (2^-52 of the populations' size over a deviation of 1e-3: 1e-11)
LARGE = {"fp32": [(1280, 1050), (256, 5203), (8192, 161)], "fp64": [(1024, 800), (64 * 13, 1001), (8192, 101)]}


@pytest.mark.parametrize("viscoelastic", [False, True])
@pytest.mark.parametrize("precision,nx,ny", [(p, *q) for p in LARGE for q in LARGE[p]])
def test_large_two_step_equals_one_step(precision, nx, ny, viscoelastic):
    c = [spec(nx, ny, wall_velocity=1e-3 if ny % 2 else 0.0)]
    a, b = (run(c, precision, 8, [16, 1], sps, viscoelastic) for sps in (0, 1))
    for p, q in zip(a[0], b[0]):
        scale = np.abs(q - (workloads.REST_WEIGHTS[:, None, None] if q.shape[0] == 9 and q.ndim == 3 else 0)).max()
        err = np.abs(p - q).max() / scale
        print(f"{precision} {nx}x{ny} viscoelastic {viscoelastic}: {err:.2e}", flush=True)
        assert err <= (2e-4 if precision == "fp32" else 1e-9 if q.ndim == 2 else 1e-11)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("viscoelastic", [False, True])
@pytest.mark.parametrize("wall", [{}, dict(wall_velocity=1e-2, top_wall="zou_he")])
def test_large_steps_off_block_boundaries(precision, viscoelastic, wall):
    """Above the boxes' limits steps outside whole blocks go two per launch, a
    last odd one alone: the same bits however the steps are split over calls."""
    c = [spec(1024, 1100, **wall)]
    a = run(c, precision, 8, [16], 0, viscoelastic)
    for steps in ([3, 5, 1, 7], [1] * 16):
        assert_same(a, run(c, precision, 8, steps, 0, viscoelastic), (precision, viscoelastic, steps))


# bounds of the pressure-drive state parity (50 x 1e-12 and 50 x 2e-6 of the
# state's deviation from rest after some tens of steps)
@pytest.mark.parametrize("precision,tol", [("fp32", 1e-4), ("fp64", 5e-11)])
@pytest.mark.parametrize("nx,ny,steps", [(2, 3, 30), (16, 64, 30), (64, 32, 30), (33, 1100, 20), (700, 5, 30),
                                         (1030, 1030, 6)])
def test_pressure_boxes_match_oracle(orc, precision, tol, nx, ny, steps):
    """The boundary columns inside the box launch: a channel of one box, boxes
    that store one of the two columns or neither, columns taller than a
    workgroup; and (1030 x 1030, above the boxes' limit) the column pass over
    more rows than it takes at once. The drive ends inside the run, which is
    split off the block boundaries."""
    from paper_1310_7450_amd import Solver
    c = spec(nx, ny, force=0.0, pressure_gradient=1e-6, nn_pressure=False, t_startup=steps - 3)
    pops, P = workloads.random_state(nx, ny, seed=nx + 5 * ny)
    o = orc.Channel(nx, ny, 0.0, tau_lb=c.tau_lb, G=c.G, tau0=c.tau0, gamma_c=c.gamma_c, eps=c.eps,
                    visc_split=c.visc_split, t_startup=c.t_startup, nn_pressure=False,
                    pressure_gradient=c.pressure_gradient)
    o.set_state(pops, P, t=0)
    with Solver([c], precision=precision, obs_every=4) as s:
        s.set_state(0, pops, P, 0)
        for n in (steps - 5, 5):
            s.step(n)
        o.run(steps)
        err = np.abs(s.get_state(0)[0] - o.n).max() / np.abs(o.n - workloads.REST_WEIGHTS[:, None, None]).max()
    print(f"{precision} {nx}x{ny}: {err:.2e}", flush=True)
    assert err < tol


@pytest.mark.parametrize("nx,ny", [(2, 400), (3, 300), (2, 512), (24, 300), (24, 513), (40, 1000), (4, 17000)])
def test_pressure_column_sum_has_one_order(nx, ny):
    """FP64 columns of more than 256 rows: the density of an inlet or outlet
    column is summed in one order, whatever workgroup size the plan of the
    handle's channels picks and whether a launch takes one step or many."""
    kw = dict(force=0.0, pressure_gradient=1e-6, nn_pressure=False)
    c = spec(nx, ny, **kw)
    others = [[], [spec(300, 11)], [spec(700, 900, **kw)], [spec(64, 32, **kw)] * 40,
              [spec(16 + i, 260 + 9 * i, **kw) for i in range(30)]]
    first = run([c], "fp64", 40, [80], 0)
    for o in others:
        for steps in ([80], [1] * 45 + [35]):
            assert_same(first, run([c] + o, "fp64", 40, steps, 0)[:1], (nx, ny, len(o), steps))


@pytest.mark.parametrize("viscoelastic", [False, True])
@pytest.mark.parametrize("precision,nx,ny", [(p, *q) for p in LARGE for q in LARGE[p]])
def test_large_two_step_same_bits(precision, nx, ny, viscoelastic):
    """What lets steps be split over calls in any way: two steps of a launch
    round as two launches do, blocks and pairs off their boundaries alike."""
    c = [spec(nx, ny, wall_velocity=1e-3 if ny % 2 else 0.0)]
    a, b = (run(c, precision, 8, [16, 1, 6], sps, viscoelastic) for sps in (0, 1))
    assert_same(a, b, (precision, nx, ny, viscoelastic))


@pytest.mark.parametrize("wall", [{}, dict(wall_velocity=0.02)])
def test_stress_force_boxes_same_bits(wall):
    kw = dict(nn_pressure=False, t_startup=31, **wall)
    shapes = [(1, 1), (3, 1), (5, 2), (8, 40), (64, 3), (8, 400), (200, 20), (143, 43), (37, 113), (1000, 9),
              (500, 300), (600, 300)]
    for case in [[q] for q in shapes] + [shapes[3:8]]:
        c = [spec(nx, ny, **kw) for nx, ny in case]
        a, b = (run(c, "fp64", 40, [80, 7, 1], sps, stress_force=True) for sps in (0, 1))
        assert_same(a, b, case)


# channels whose single steps, or all off the block boundaries, leave the boxes
# that take their blocks
SPLIT = [("fp32", 1024, 600), ("fp32", 1024, 850), ("fp32", 3000, 750), ("fp64", 512, 512), ("fp64", 1024, 512),
         ("fp64", 500, 500), ("fp64", 300, 700)]


@pytest.mark.parametrize("viscoelastic", [False, True])
@pytest.mark.parametrize("precision,nx,ny", SPLIT)
def test_steps_split_over_calls_in_any_way(precision, nx, ny, viscoelastic):
    c = [spec(nx, ny, wall_velocity=1e-3, t_startup=11)]
    a = run(c, precision, 12, [24], 0, viscoelastic)
    for steps in ([1] * 24, [5, 7, 1, 11], [13, 11], [12, 3, 9]):
        assert_same(a, run(c, precision, 12, steps, 0, viscoelastic), (precision, nx, ny, viscoelastic, steps))
