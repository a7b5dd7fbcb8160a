"""The launches of multi-step calls, from the host code alone (no GPU)."""
import pytest

from hip_recorder import launches


def pairs_of_buffers(rows):
    return [(r[3], r[4]) for r in rows]


def test_captured_even_calls_end_where_they_start():
    """A graph of an even number of steps is replayed from the buffer that held
    the state at capture, so it has to end there; an odd call changes buffers.
    Every launch reads what the one before it wrote."""
    runs = launches("""
out = []
for dims in ((8, 8, 8), (9, 11, 13, 2), (32, 32, 16), (32, 32, 32), (8, 60, 60), (8, 9, 8, 30), (64, 64, 64)):
    for storage in ("fp64", "fp32"):
        for wall in (0, 1):
            h = handle3(*dims, storage=storage, wall=wall)
            for n in range(1, 12):
                t = time_of(L3.cmlbm_get_time, h)
                rec(capture=1)
                assert L3.cmlbm_step(h, n, STREAM) == 0
                out.append([dims, storage, n, time_of(L3.cmlbm_get_time, h) - t, seen()])
""")
    assert any("k_tile<double, 2" in r[0] for *_, rows in runs for r in rows)
    for dims, storage, n, steps, rows in runs:
        bufs = pairs_of_buffers(rows)
        assert steps == n
        assert all(a[1] == b[0] for a, b in zip(bufs, bufs[1:]))
        assert (bufs[0][0] == bufs[-1][1]) == (n % 2 == 0), (dims, storage, n)


def test_captured_even_calls_of_the_plane_solver_end_where_they_start():
    runs = launches("""
out = []
for dims in ((1, 1), (8, 8), (64, 64), (300, 211), (64, 70000), (1025, 1100), (4096, 1100), (3001, 1500), (8192, 8192)):
    for storage in ("fp64", "fp32", "fp16"):
        h = handle2(*dims, storage=storage)
        for n in list(range(1, 26)) + [100, 101]:
            t = time_of(L2.cmlbm2d_get_time, h)
            rec(capture=1)
            assert L2.cmlbm2d_step(h, n, STREAM) == 0
            out.append([dims, storage, n, time_of(L2.cmlbm2d_get_time, h) - t, seen()])
""")
    names = {r[0].split("<")[0] for *_, rows in runs for r in rows}
    assert names == {"k2_step", "k2_march", "k2_tile"}
    for dims, storage, n, steps, rows in runs:
        bufs = pairs_of_buffers(rows)
        assert steps == n
        assert all(a[1] == b[0] for a, b in zip(bufs, bufs[1:]))
        assert (bufs[0][0] == bufs[-1][1]) == (n % 2 == 0), (dims, storage, n)


def test_a_launch_that_fails_inside_the_moment_path_ends_the_state():
    """Between the first and the last step of such a call a buffer holds nine
    numbers per cell: if a launch fails there, nothing may read it as
    populations.  A failure of the first launch leaves the state as it was, and
    so does any failure of a call whose every launch writes populations."""
    codes = launches("""
out = []
for dims, fail in (((64, 64, 64), 0), ((64, 64, 64), 1), ((64, 64, 64), 3), ((48, 40, 40), 2)):
    h = handle3(*dims)
    rec(fail=fail)
    first = L3.cmlbm_step(h, 5, None)
    launched = len(seen())
    rec()
    after = [L3.cmlbm_step(h, 1, None), L3.cmlbm_moments(h, F, None, 0, None), L3.cmlbm_populations(h, F, None),
             L3.cmlbm_save_state(h, F, 1 << 40, None)]
    again = L3.cmlbm_init(h, None, None, 0, None)
    out.append([first, launched, after, again, L3.cmlbm_step(h, 5, None)])
""")
    EHIP, ESTATE = -3, -5
    assert codes == [[EHIP, 0, [0] * 4, 0, 0], [EHIP, 1, [ESTATE] * 4, 0, 0], [EHIP, 3, [ESTATE] * 4, 0, 0],
                     [EHIP, 2, [0] * 4, 0, 0]]


def test_calls_between_replays_keep_the_buffers():
    """Once any call on a lattice has been captured, ordinary calls of an even
    number of steps end in the buffer they start in as well: a graph goes on from
    the buffers of its capture.  Until then they take the fewest launches."""
    runs = launches("""
out = []
firsts3 = [lambda h: L3.cmlbm_step(h, 2, STREAM), lambda h: L3.cmlbm_moments(h, F, None, 0, STREAM),
           lambda h: L3.cmlbm_populations(h, F, STREAM), lambda h: L3.cmlbm_step_velocity(h, F, 0, STREAM),
           lambda h: L3.cmlbm_save_state(h, F, 1 << 40, STREAM), lambda h: L3.cmlbm_restore_state(h, F, 1 << 40, STREAM),
           lambda h: L3.cmlbm_load_populations(h, F, STREAM)]
firsts2 = [lambda h: L2.cmlbm2d_step(h, 1, STREAM), lambda h: L2.cmlbm2d_moments(h, F, None, 0, STREAM),
           lambda h: L2.cmlbm2d_populations(h, F, STREAM), lambda h: L2.cmlbm2d_load_populations(h, F, STREAM)]
for make, step, firsts in ((lambda: handle3(8, 9, 8, 30), L3.cmlbm_step, firsts3),
                           (lambda: handle2(2048, 2048), L2.cmlbm2d_step, firsts2)):
    for first in firsts:
        h = make()
        assert step(h, 2, STREAM) == 0
        rec()
        assert step(h, 2, STREAM) == 0
        before = len(seen())
        rec(capture=1)
        assert first(h) == 0
        rec(capture=0)
        rows = []
        for n in (2, 4, 6, 8):
            rec()
            assert step(h, n, None) == 0
            rows.append(seen())
        out.append([before, rows])
""")
    assert len(runs) == 11
    for before, calls in runs:
        assert before == 1
        for rows in calls:
            assert len(rows) % 2 == 0 and rows[0][3] == rows[-1][4]


def conv_launches(cases):
    """The kernel, grid and block of forward convolutions ((n, d, h, w), input and output channels)."""
    return launches(f"""
out = []
for dims, cin, cout in {cases!r}:
    g = NN.geom(*dims)
    rec()
    assert LN.cmnn_conv3d_fwd(ctypes.byref(g), A, cin, B, None, cout, 0, S, None) == 0
    out += [r[:3] for r in seen()]
""")


def test_convolution_launches_have_fewer_than_2_to_the_32_work_items():
    """A launch's extents count work-items in 32 bits.  The calls here fit a
    288 GiB device (the last: 17 GB in, 275 GB out)."""
    cases = [((1024, 32, 32, 128), 32, 1024), ((1024, 32, 28, 128), 64, 1024), ((2048, 16, 4, 1024), 64, 1024)]
    for (kernel, grid, block), case in zip(conv_launches(cases), cases):
        assert grid[0] * block < 1 << 32, (kernel, case)


# (n, d, h, w), input and output channels, kernel: both sides of every line of the dispatch's rule
CONV_ROUTES = [
    ((2, 3, 5, 7), 32, 64, "k_conv_fwd<4"), ((1, 4, 6, 16), 32, 96, "k_conv_fwd<2"),    # no bricks
    ((192, 4, 8, 16), 32, 32, "k_conv_rows"), ((191, 4, 8, 16), 64, 32, "k_conv_few"),  # 192 row workgroups
    ((16, 8, 8, 16), 32, 64, "k_conv_tile<1"), ((16, 8, 12, 16), 32, 64, "k_conv_few"),  # one chunk: 128, 192 workgroups
    ((64, 8, 4, 16), 96, 64, "k_conv_few"), ((65, 8, 4, 16), 96, 64, "k_conv_tile<2"),  # 256, 260 workgroups
    ((65, 8, 4, 16), 64, 64, "k_conv_few"), ((16, 32, 28, 64), 128, 128, "k_conv_few"),  # whole lines of weights
    ((16, 32, 28, 64), 32, 32, "k_conv_tile<2"), ((16, 32, 28, 64), 96, 64, "k_conv_tile<4"),
    ((16, 32, 28, 64), 32, 96, "k_conv_tile<6"), ((16, 32, 28, 64), 96, 192, "k_conv_tile<6"),
]


# the large batches and the small ones of test_gpu_conv_routes.py
CONV_ROUTES += [
    ((32, 16, 4, 64), 32, 64, "k_conv_tile<4"), ((1, 16, 4, 64), 32, 64, "k_conv_tile<1"),
    ((33, 16, 4, 64), 96, 96, "k_conv_tile<6"), ((2, 16, 4, 64), 96, 96, "k_conv_few"),
    ((1, 4, 4, 16), 64, 32, "k_conv_few"), ((4, 8, 12, 16), 32, 64, "k_conv_tile<1"),
]


def test_convolution_kernels_by_size():
    got = conv_launches([c[:3] for c in CONV_ROUTES])
    for (kernel, *_), case in zip(got, CONV_ROUTES):
        assert kernel.startswith(case[3]), (kernel, case)


def box_launches(cases):
    """Per case ((nx, ny, nz, nbatch), storage, wall, field, steps): the kernels of one call."""
    return launches(f"""
out = []
for dims, storage, wall, field, n in {cases!r}:
    h = handle3(*dims, storage=storage, wall=wall, field=field)
    rec()
    assert L3.cmlbm_step(h, n, None) == 0
    out.append([r[0] for r in seen()])
""")


# three steps a launch up to a workgroup a CU; two up to that, and up to two workgroups a CU where
# k_step has more than 1024 waves or FP32 a wall; FP32 then ends a call on three, and takes three on
# rows with too many tiles of two; one beyond
TILE_ROUTES = [
    ((32, 32, 16, 1), 5, ["k_tile 3", "k_tile 2"]), ((32, 32, 20, 1), 5, ["k_step"] * 5),
    ((32, 32, 32, 1), 3, ["k_step"] * 3), ((22, 36, 31, 1), 6, ["k_tile 2", "k_tile 2", "k_tile 2"]),
    ((8, 60, 60, 1), 5, ["k_tile 2", "k_tile 2", "k_step"]), ((11, 42, 51, 1), 7, ["k_step"] * 7),
    ((8, 9, 8, 30), 3, ["k_tile 2", "k_step"]), ((8, 9, 8, 30), 6, ["k_tile 2", "k_tile 2", "k_tile 2"]),
    ((9, 11, 13, 2), 7, ["k_tile 3", "k_tile 3", "k_step"]), ((32, 32, 36, 1), 4, ["k_step"] * 4),
    ((7, 8, 8, 1), 3, ["k_step"] * 3), ((8, 8, 8, 1), 1, ["k_step"]),
]
TILE_ROUTES_FP32 = {((8, 60, 60, 1), 5): ["k_tile 2", "k_tile 3"], ((8, 9, 8, 30), 3): ["k_tile 3"],
                    ((11, 42, 51, 1), 7): ["k_tile 3", "k_tile 3", "k_step"]}
TILE_ROUTES_FP32_WALL = {((32, 32, 20, 1), 5): ["k_tile 2", "k_tile 3"], ((32, 32, 32, 1), 3): ["k_tile 3"]}


@pytest.mark.parametrize("storage", ["fp64", "fp32"])
@pytest.mark.parametrize("wall", [0, 1])
def test_kernels_of_small_lattices_by_size(storage, wall):
    got = box_launches([(dims, storage, wall, 0, n) for dims, n, _ in TILE_ROUTES])
    other = {**TILE_ROUTES_FP32, **(TILE_ROUTES_FP32_WALL if wall else {})} if storage == "fp32" else {}
    for kernels, (dims, n, want) in zip(got, TILE_ROUTES):
        short = [k.split("<")[0] + (" " + k.split(", ")[1] if k.startswith("k_tile") else "") for k in kernels]
        assert short == other.get((dims, n), want), (dims, n)


# (nx, ny, nz, nbatch), storage, wall, field, steps; whether the call goes through the nine numbers
MARCH_ROUTES = [
    ((64, 64, 64, 1), "fp64", 1, 0, 2, False), ((64, 64, 64, 1), "fp64", 1, 0, 10, True),
    ((64, 64, 64, 1), "fp64", 1, 1, 10, False), ((128, 128, 128, 1), "fp64", 1, 1, 3, True),
    ((80, 80, 80, 1), "fp64", 1, 1, 10, False), ((80, 80, 80, 1), "fp64", 0, 1, 2, True),
    ((8, 320, 320, 1), "fp64", 1, 1, 10, False), ((8, 320, 320, 1), "fp64", 0, 0, 2, True),
    ((16, 256, 256, 1), "fp64", 1, 0, 2, False), ((16, 256, 256, 1), "fp32", 1, 1, 2, True),
    ((64, 64, 64, 1), "fp32", 0, 0, 10, False), ((80, 80, 80, 1), "fp32", 1, 1, 2, True),
    ((5, 11, 40, 512), "fp64", 0, 0, 10, False), ((5, 11, 40, 64), "fp32", 0, 1, 2, False),
    ((256, 256, 256, 1), "fp32", 1, 1, 2, True), ((256, 256, 256, 1), "fp64", 1, 1, 2, True),
]


def test_moment_path_by_size():
    got = box_launches([c[:5] for c in MARCH_ROUTES])
    for kernels, (*case, march) in zip(got, MARCH_ROUTES):
        n = case[-1]
        if march:
            assert kernels[0].startswith("k_step<") and kernels[0].endswith(", 1>"), case  # nine numbers out
            assert all(k.startswith("k_march<") for k in kernels[1:]), case
            assert [k.endswith("true>") for k in kernels[1:]] == [False] * (n - 2) + [True], case  # populations last
        else:
            assert len(kernels) == n and all(k.startswith("k_step<") for k in kernels), case


def test_tile_rows_of_the_moment_kernel():
    """FP64 tiles of 8 rows; FP32 12, or 6 for few rows and for lattices that do
    not give every CU a tile of 12."""
    cases = [((256, 256, 1, 1), "mom32", 6), ((64, 64, 64, 1), "mom32", 6), ((64, 64, 16, 1), "mom32", 6),
             ((512, 512, 1, 1), "mom32", 12), ((200, 200, 8, 1), "mom32", 12), ((96, 96, 96, 1), "mom32", 12),
             ((256, 256, 256, 1), "mom32", 12), ((96, 20, 96, 8), "mom32", 6), ((64, 32, 32, 16), "fp32", 12),
             ((64, 32, 32, 16), "fp64", 8)]
    got = box_launches([(dims, storage, 0, 0, 2) for dims, storage, _ in cases])
    for kernels, (dims, storage, rows) in zip(got, cases):
        kind = "double" if storage == "fp64" else "float"
        assert kernels[1].startswith(f"k_march<{kind}, {rows}, "), (dims, kernels)


def test_population_storage_keeps_its_tile_rows():
    """The choice of 6 rows on small lattices is moment storage's: 65^3 in FP32
    takes tiles of 12 (183 us for ten steps; with tiles of 6 not chosen, 195)."""
    (kernels,) = box_launches([((65, 65, 65, 1), "fp32", 0, 0, 10)])
    assert kernels[1].startswith("k_march<float, 12, ")


def test_lattices_of_the_schedule_tests_take_the_moment_path():
    """Of test_gpu_march_schedule.py: every kind of lattice, and the blocked order,
    whose grid is rounded up beyond the tiles, on the first two."""
    blocked = {"fp64": (120, 122, 6, 66), "fp32": (120, 190, 6, 66)}
    tiles = {"fp64": 2 * 16 * 66, "fp32": 2 * 16 * 66}
    runs = launches(f"""
out = []
for storage, dims in list({blocked!r}.items()) + [(s, (40, 60, 40, 8)) for s in ("fp64", "fp32")]:
    for wall in (0, 1):
        for field in (0, 1):
            for n in (6, 7):
                h = handle3(*dims, storage=storage, wall=wall, field=field)
                rec()
                assert L3.cmlbm_step(h, n, None) == 0
                out.append([storage, list(dims), n, seen()])
""")
    for storage, dims, n, rows in runs:
        assert [r[0].split("<")[0] for r in rows] == ["k_step"] + ["k_march"] * (n - 1), (storage, dims)
        if tuple(dims) == blocked[storage]:
            assert rows[1][1][0] > tiles[storage] and rows[1][1][0] % 256 == 0


def plane_launches(cases):
    """Per case ((nx, ny), storage, steps): the kernels of one call of the plane solver."""
    return launches(f"""
out = []
for dims, storage, n in {cases!r}:
    h = handle2(*dims, storage=storage)
    rec()
    assert L2.cmlbm2d_step(h, n, None) == 0
    out.append([r[0] for r in seen()])
""")


def test_planes_of_the_long_pass_tests_take_them():
    """Of test_gpu_march2d_eight.py and test_gpu_nonfinite.py."""
    cases = [(d, "fp32", n) for d in ((8192, 1750), (5000, 3750), (128, 70000)) for n in (8, 21)]
    for kernels in plane_launches(cases):
        assert any(k.startswith("k2_march<1, 2, 8,") for k in kernels)
    cases = [((300, 211), 7, "k2_tile"), ((1025, 1100), 4, "k2_march<{}, 1, 4,"), ((4096, 1100), 6, "k2_march<{}, {}, 6,"),
             ((8192, 1750), 8, "k2_march<{}, {}, 8,")]
    for storage, st, v in (("fp64", 0, 1), ("fp32", 1, 2)):
        for kernels, (dims, n, want) in zip(plane_launches([(d, storage, n) for d, n, _ in cases]), cases):
            assert any(k.startswith(want.format(st, v)) for k in kernels), (dims, storage, kernels)


def test_passes_take_the_steps_that_they_count():
    """Every k2_march launch is the kernel of as many steps as the call advances by,
    on odd rows (one FP32 cell a lane, six at most) too."""
    dims = [(3001, 1500), (5001, 3750), (8191, 2048), (4096, 1100), (1025, 1100), (129, 70000)]
    runs = launches(f"""
out = []
for dims in {dims!r}:
    for storage in ("fp64", "fp32"):
        h = handle2(*dims, storage=storage)
        for n in (2, 4, 6, 8, 16, 40):
            rec()
            assert L2.cmlbm2d_step(h, n, None) == 0
            out.append([dims, storage, n, [r[0] for r in seen()]])
""")
    for dims, storage, n, kernels in runs:
        if any(k.startswith("k2_tile") for k in kernels):
            continue
        steps = [int(k.split(", ")[2]) if k.startswith("k2_march") else 1 for k in kernels]
        assert sum(steps) == n, (dims, storage, kernels)
        if storage == "fp32" and dims[0] % 2:
            assert max(steps) <= 6


@pytest.mark.parametrize("cus", [64, 256])
def test_plane_passes_are_sized_for_the_compute_units(cus):
    """k2_march's waves fill the SIMDs of the lattice's device, as many each as its
    registers leave room for."""
    runs = launches(f"""
out = []
rec(cus={cus})
for dims in ((4096, 4096), (8192, 8192)):
    h = handle2(*dims, storage="fp64")
    rec(cus={cus})
    assert L2.cmlbm2d_step(h, 8, None) == 0
    out.append(seen())
""")
    for rows in runs:
        kernel, grid, block = rows[0][:3]
        assert kernel.startswith("k2_march<0, 1, ")
        assert grid[0] * block // 64 <= {"2": 4, "4": 3, "6": 2, "8": 2}[kernel.split(", ")[2]] * 4 * cus
