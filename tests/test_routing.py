"""Which launches advance which channels, on the CPU: the host runtime linked
with stand-ins for HIP and for its launchers (host_routing_driver.cpp), which
check that every step of every channel is taken once, from the right buffer,
and with the pressure drive's boundary applied once."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="session")
def route(tmp_path_factory):
    """route(precision, K, steps, channels, ...) -> per channel a dict of
    steps by launcher and "most", the most steps of one launch."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc) and shutil.which("hipcc") is None:
        pytest.skip("hipcc not available")
    exe = tmp_path_factory.mktemp("routing") / "host_routing"
    csrc = os.path.join(ROOT, "paper_1310_7450_amd", "csrc")
    cmd = [hipcc, "--offload-arch=gfx950", "-O1", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
           "-packed-fp32-ops", "-I", os.path.join(ROOT, "include"), "-I", csrc, os.path.join(csrc, "lb_runtime.hip"),
           os.path.join(ROOT, "tests", "host_routing_driver.cpp"), "-o", str(exe)]
    build = subprocess.run(cmd, capture_output=True, text=True, timeout=600)
    assert build.returncode == 0, build.stderr[-2000:]

    def run(precision, K, steps, channels, viscoelastic=0, stress_force=0, steps_per_sweep=0):
        args = [f"{nx},{ny}," + ",".join(str(int(f in flags)) for f in ("pressure", "wall", "zou_he"))
                for nx, ny, *flags in channels]
        r = subprocess.run([str(exe), precision, str(K), str(viscoelastic), str(stress_force), str(steps_per_sweep),
                            ",".join(map(str, steps)), *args], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]
        return [{k: int(v) for k, v in (w.split("=") for w in line.split()[2:])}
                for line in r.stdout.splitlines() if line.startswith("channel")]

    return run


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_pressure_channel_beyond_the_boxes_keeps_its_boundary(route, precision):
    """A pressure-driven channel too large for the boxes' 32-bit slots beside a
    short one that takes many steps per launch: the column pass follows each of
    its steps, in whole blocks too."""
    large, small = route(precision, 20, [40, 3, 1, 60], [(1 << 20, 410, "pressure"), (64, 32, "pressure")])
    assert large["column_pass"] == 104 and "boxes" not in large
    assert small["boxes"] == 104 and small["most"] > 1


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("K,steps", [(20, [40, 3, 1, 60]), (2, [7]), (6, [5, 13]), (100, [250, 1, 49])])
@pytest.mark.parametrize("viscoelastic", [0, 1])
def test_every_step_once(route, precision, K, steps, viscoelastic):
    """Channels of every route in one handle, and each alone: narrow, aligned
    and other widths below and above the boxes' limits, walls, the pressure
    drive short, tall and above its limit."""
    chans = [(8, 40, "wall"), (512, 40), (300, 11), (600, 3000), (1024, 2000, "zou_he"), (64, 20000), (32, 9),
             (64, 32, "pressure"), (24, 300, "pressure")]
    for case in [chans, chans + [(1100, 1000, "pressure")], chans[:3] + chans[6:7], chans[7:]] + [[c] for c in chans]:
        route(precision, K, steps, case, viscoelastic)
        route(precision, K, steps, case, viscoelastic, steps_per_sweep=1)


@pytest.mark.parametrize("precision,shape,boxes", [
    ("fp64", (100, 5000), True), ("fp64", (100, 7500), False), ("fp64", (16, 10000), True),
    ("fp64", (16, 15800), False), ("fp64", (4, 31600), True), ("fp64", (4, 100000), False),
    ("fp32", (30, 30000), True), ("fp32", (4, 100000), True)])
def test_tall_pressure_channels_keep_the_column_pass(route, precision, shape, boxes):
    """Boxes of a tall channel would each sum whole columns: strips and the
    column pass take it, also beside a short channel in boxes."""
    for case in [[(*shape, "pressure")], [(*shape, "pressure"), (64, 32, "pressure")]]:
        tall, *rest = route(precision, 20, [40, 3], case)
        assert ("boxes" in tall) == boxes and all(c["boxes"] == 43 for c in rest)
        assert tall.get("column_pass", 0) == (0 if boxes and precision == "fp64" else 43)


@pytest.mark.parametrize("precision,shape,viscoelastic,single", [
    ("fp32", (512, 512), 0, "boxes"), ("fp32", (1024, 600), 0, "sweep"), ("fp32", (1024, 600), 1, "boxes"),
    ("fp64", (256, 128), 0, "boxes"), ("fp64", (512, 512), 0, "tiles"), ("fp64", (1000, 100), 0, "tiles"),
    ("fp64", (300, 100), 0, "boxes"), ("fp64", (4000, 2000), 1, "tiles"), ("fp64", (8, 262144), 0, "boxes"),
    ("fp64", (66, 4000), 0, "boxes")])
def test_blocks_of_one_step_plans(route, precision, shape, viscoelastic, single):
    """Half a block without a divisor that pays (1, 503): boxes of one step
    replace the one-step sweeps only where they are faster; blocks of many
    divisors keep the boxes."""
    for K in (2, 1006):
        c, = route(precision, K, [2 * K], [shape], viscoelastic)
        assert c[single] == 2 * K and c["most"] == 1
    c, = route(precision, 1000, [1000], [shape], viscoelastic)
    assert c["boxes"] == 1000 and c["most"] > 1


@pytest.mark.parametrize("precision,shape,single,several", [
    ("fp32", (512, 512), "boxes", "boxes"), ("fp32", (1024, 700), "sweep", "boxes"),
    ("fp32", (1024, 850), "sweep", "sweep"), ("fp32", (4000, 1000), "sweep", "boxes"),
    ("fp64", (256, 256), "boxes", "boxes"), ("fp64", (512, 512), "tiles", "boxes"),
    ("fp64", (1024, 512), "tiles", "tiles"), ("fp64", (500, 500), "tiles", "boxes")])
def test_steps_off_the_block_boundaries(route, precision, shape, single, several):
    """Single steps, and runs of some, by the path that is faster there."""
    c, = route(precision, 1000, [1] * 10, [shape])
    assert c[single] == 10
    c, = route(precision, 1000, [500], [shape])
    assert c[several] >= 498


def test_gpu_tests_reach_the_routes_they_name(route):
    """The handles of the two-step tests above the boxes' limits take the
    kernels those tests are about, the mixed ones every route."""
    from test_gpu_two_step import ABOVE, MIXED
    for (precision, kind), shapes in ABOVE.items():
        name = "two_step" if kind == "streamed" else kind
        for ve in (0,) if kind == "narrow_two_step" else (0, 1):
            chans = [(nx, ny, *(("wall",), ("wall", "zou_he"))[i % 2]) if ny > 1 else (nx, ny)
                     for i, (nx, ny) in enumerate(shapes)]
            for c in route(precision, 8, [16, 3, 5, 1, 2], chans, ve):
                assert c[name] >= 16 and "boxes" not in c
    for precision, shapes in MIXED.items():
        for more in ([], [(1100, 1000, "pressure")]):
            taken = set().union(*route(precision, 8, [8, 16, 3, 5, 7], shapes + more))
            assert {"boxes", "two_step", "narrow_two_step", "column_pass"} <= taken
            assert ("tiles" if precision == "fp64" else "sweep") in taken


def test_narrow_channels_beyond_the_boxes_step_singly(route):
    c, = route("fp32", 8, [8, 3], [(16, 27_000_000)])
    assert c["sweep"] == 11


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_rows_beyond_32_bit_slots_step_singly(route, precision):
    """The two-step strips address a row's slots by 32 bits: up to 429,496,729
    columns."""
    widest = (2 ** 32 // 10) // 256 * 256
    c, = route(precision, 8, [8, 3], [(widest, 1)])
    assert c["two_step"] == 10
    c, = route(precision, 8, [8, 3], [(widest + 256, 1)])
    assert c["sweep"] == 11


@pytest.mark.parametrize("precision,shapes,K,boxes", [
    ("fp64", [(2000, 64)], 1000, True), ("fp64", [(4000, 64)], 1000, False), ("fp64", [(1000, 1000)], 1000, True),
    ("fp64", [(64, 64)] * 100, 1000, False), ("fp64", [(16000, 40)], 1000, True), ("fp64", [(16000, 40)], 1006, False),
    ("fp64", [(8, 100)] * 300, 1000, True), ("fp32", [(4000, 64)], 1000, True), ("fp32", [(4096, 200)], 1000, False),
    ("fp32", [(512, 512)], 1000, True), ("fp32", [(64, 64)] * 100, 1000, True)])
def test_pressure_boxes_only_where_faster(route, precision, shapes, K, boxes):
    """Wide channels too tall for many steps per launch keep the sweeps and the
    column pass; short ones beside them their boxes."""
    chans = [(*s, "pressure") for s in shapes]
    for c in route(precision, K, [K, 3], chans):
        assert ("boxes" in c) == boxes
    *_, short = route(precision, 1000, [1000, 3], chans + [(64, 32, "pressure")])
    assert "boxes" in short


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_steps_of_two_box_lists(route, precision):
    """Off the block boundaries a handle of short pressure-driven and other small
    channels steps in both kinds of boxes, not in a sweep per width."""
    chans = [(8, 40), (300, 11), (16, 9), (64, 32, "pressure"), (24, 300, "pressure")]
    for case in (chans, chans[:4]):
        for c in route(precision, 1000, [1, 7, 40], case):
            assert c["boxes"] == 48


def test_tall_pressure_channels_together(route):
    """What the boxes of several tall FP64 channels would read of their columns
    adds up: once it is too much, all of them take the column pass."""
    one = route("fp64", 20, [20], [(100, 5000, "pressure")])
    assert one[0]["boxes"] == 20
    for c in route("fp64", 20, [20], [(100, 5000, "pressure"), (80, 5000, "pressure")]):
        assert c["column_pass"] == 20 and "boxes" not in c
    *tall, short = route("fp64", 20, [20], [(100, 5000, "pressure"), (80, 5000, "pressure"), (24, 30, "pressure")])
    assert all("boxes" not in c for c in tall) and short["boxes"] == 20
