"""Which launches calls of the library make (tests/launches.py; no GPU)."""
import pytest

from launches import record


@pytest.mark.parametrize("dtype,d_dead,every", [("f32", 0.0, 7), ("f32", 0.0, 8), ("f32", 3e-3, 8),
                                                ("f64", 3e-3, 5), ("f64", 0.0, 5)])
@pytest.mark.parametrize("shape", [(0, 0, 0), (1, 0, 0), (2, 40, 2)])
def test_a_segment_that_fits_a_march_is_one_pass(dtype, d_dead, every, shape):
    """Up to the deepest march, recorded runs write each segment straight into
    the next checkpoint in one pass, whatever the context's steps per pass."""
    if shape[2] == 2 and dtype == "f64":
        shape = (2, 40, 1)
    result = record(f'''
h = context(1536, 1100, {dtype!r}, {d_dead})
assert lib.sslbm_set_launch(h, ctypes.byref(Launch(*{shape}))) == 0
steps = 3 * {every} + 2
one = passes(lambda: lib.sslbm_run_checkpointed(h, rho, scratch, steps, {every}, extra, None))
result = [one, [l[4:] for l in launched()]]
''')
    kinds, ends = result
    assert [k[:2] for k in kinds] == [["copy", None]] + 3 * [["march", every]] + [["march", 2]]
    scratch = 2 << 40
    assert all(scratch not in e for e in ends)  # scratch is not touched
    assert all(ends[i][1] == ends[i + 1][0] for i in range(1, 4))
    assert ends[-1][1] == 1 << 40  # the last segment ends in rho


@pytest.mark.parametrize("dtype", ["f32", "f64"])
@pytest.mark.parametrize("every", [1, 2, 3, 4, 5, 7, 11, 23])
def test_tile_segments_take_the_fewest_passes(dtype, every):
    """On small grids too a segment needs no even number of passes, and the
    passes' shape is worked out once a call, not once a segment."""
    result = record(f'''
h = context(128, 128, {dtype!r})
kinds = passes(lambda: lib.sslbm_run_checkpointed(h, rho, scratch, 40 * {every}, {every}, extra,
                                                  None))
result = [kinds, rec.rec_queries()]
''')
    kinds, queries = result
    if every == 2:
        assert [k[0] for k in kinds] == ["copy"] + 20 * ["mid"]
    else:
        assert {k[0] for k in kinds[1:]} == {"tile"}
        # FP64 tiles of one row a lane hold at most 7 steps
        assert (len(kinds) - 1) % 40 == 0 and (len(kinds) - 1) // 40 <= -(-every // 7)
        assert queries < 20  # of the device, one a plan: 40 segments


# (nx, ny), kernels of a run: tiles where they are faster, the march on grids
# a few cells high, long ones a few cells wide, and where it just fills the GPU
ROUTES = {
    "f32": [((1, 1), "tile"), ((128, 128), "tile"), ((1024, 1024), "tile"), ((20000, 8), "tile"),
            ((16, 12500), "tile"), ((64, 6875), "tile"), ((1180, 1180), "tile"),
            ((262144, 1), "march"), ((70000, 2), "march"), ((131072, 8), "march"),
            ((1, 440000), "march"), ((1300, 1300), "march")],
    "f64": [((1, 1), "tile"), ((128, 128), "tile"), ((512, 512), "tile"), ((200, 2000), "tile"),
            ((12500, 16), "tile"), ((16, 4375), "tile"), ((262144, 1), "march"),
            ((35000, 2), "march"), ((32768, 8), "march"), ((1, 70000), "march"),
            ((4, 100000), "march"), ((700, 700), "march")],
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_tiles_only_where_they_are_faster(dtype):
    """Single grids, and ensembles of one grid too large for LDS."""
    result = record(f'''
result = []
for (nx, ny), want in {ROUTES[dtype]!r}:
    h = context(nx, ny, {dtype!r})
    single = {{k[0] for k in passes(lambda: lib.sslbm_run(h, rho, scratch, 60, None))}}
    many = {{want}}
    if 5 * nx * ny * {4 if dtype == "f32" else 8} > 81920 and max(nx, ny) <= 65536:
        e = ensemble([(nx, ny)], {dtype!r})
        many = {{k[0] for k in passes(lambda: lib.sslbm_ensemble_run(e, rho, scratch, 60, 0, None))}}
    result.append([nx, ny, sorted(single), sorted(many), want])
''')
    bad = [r for r in result if r[2] != [r[4]]]
    assert not bad, bad
    # ensembles name their march kernel differently
    bad = [r for r in result if r[4] == "tile" and r[3] != ["tile"]]
    assert not bad, bad


# (nx, ny, steps) -> kernels: short runs by their own estimate, grids of few tiles
# and in FP32 thin ones as long runs
SHORT = {
    "f32": [((128, 128), 5, "tile"), ((768, 768), 2, "march"), ((768, 768), 14, "tile"),
            ((1024, 1024), 4, "march"), ((1024, 1024), 16, "tile"), ((1024, 1024), 25, "tile"),
            ((1500, 901), 7, "march"), ((3000, 200), 5, "march"), ((10000, 40), 5, "tile"),
            ((400, 400), 12, "tile")],
    "f64": [((128, 128), 12, "tile"), ((400, 400), 14, "tile"), ((670, 670), 12, "tile"),
            ((4096, 64), 2, "march"), ((670, 670), 3, "march"), ((670, 670), 60, "tile"),
            ((20000, 13), 3, "march"), ((5000, 60), 3, "march"), ((8, 12000), 4, "march"),
            ((8000, 30), 12, "tile"), ((5000, 60), 14, "tile")],
}


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_short_runs_take_the_faster_passes(dtype):
    """A single grid's run and its plan, and an ensemble of one such grid, whose
    passes all have the rows of its deepest one."""
    result = record(f'''
result = []
for (nx, ny), steps, want in {SHORT[dtype]!r}:
    h = context(nx, ny, {dtype!r})
    single = [k for k in passes(lambda: lib.sslbm_run(h, rho, scratch, steps, None))
              if k[0] != "copy"]
    n, hi, lo = ctypes.c_longlong(), ctypes.c_int(), ctypes.c_int()
    lib.sslbm_plan_run(h, steps, ctypes.byref(n), ctypes.byref(hi), ctypes.byref(lo))
    e = ensemble([(nx, ny)], {dtype!r})
    many = "tile"
    if 5 * nx * ny * {4 if dtype == "f32" else 8} > 81920:
        kinds = passes(lambda: lib.sslbm_ensemble_run(e, rho, scratch, steps, 0, None))
        many = "tile" if kinds[0][0] == "tile" else "march"
    result.append([nx, ny, steps, want, sorted({{k[0] for k in single}}), len(single) == n.value,
                   many])
''')
    bad = [r for r in result if r[4] != [r[3]] or not r[5]]
    assert not bad, bad
    one = {tuple(r[:3]): r[6] for r in result}
    if dtype == "f32":
        assert one[1500, 901, 7] == "march" and one[1024, 1024, 16] == "tile"
    else:
        assert one[670, 670, 3] == "march" and one[670, 670, 12] == "tile"


def test_marches_of_a_tuned_context_have_the_tuned_rows():
    """After a tuning that tiles won, marches (single steps, recorded runs
    every second step) run the shape that was timed, columns and rows."""
    best, rows, auto = record('''
h = context(900, 900)
step = lambda: lib.sslbm_step(h, rho, scratch, None)
passes(step)
auto = rec.rec_arg(0, 4, 0)
rec.rec_price(b"march", 6.0)
rec.rec_price(b"tile", 0.1)
best = Launch()
assert lib.sslbm_tune(h, rho, scratch, None, ctypes.byref(best)) == 0
assert {k[0] for k in passes(lambda: lib.sslbm_run(h, rho, scratch, 40, None))} == {"tile"}
assert passes(step)[0] == ("march", 1, best.cols_per_lane)
result = [best.as_dict(), rec.rec_arg(0, 4, 0), auto]
''')
    assert rows == best["rows_per_wave"] and rows != auto


def test_a_tuned_choice_of_tiles_can_be_passed_on():
    """The shape that a tuning reports, set on another context, gives that
    context the same passes, through the C ABI and the Python class."""
    a, b, march, codes, py, py_march = record('''
run = lambda c: passes(lambda: lib.sslbm_run(c, rho, scratch, 40, None))
h, other = context(1090, 1090), context(1090, 1090)
rec.rec_price(b"march", 6.0)
rec.rec_price(b"tile", 0.1)
best = Launch()
assert lib.sslbm_tune(h, rho, scratch, None, ctypes.byref(best)) == 0
assert lib.sslbm_get_tiles(h) == 1 and lib.sslbm_get_tiles(other) == 0
assert lib.sslbm_set_tiles(other, ctypes.byref(best)) == 0 and lib.sslbm_get_tiles(other) == 1
a, b = run(h), run(other)
assert lib.sslbm_set_launch(other, ctypes.byref(best)) == 0 and lib.sslbm_get_tiles(other) == 0
march = run(other)
large = context(2000, 2000)
codes = [lib.sslbm_set_tiles(large, ctypes.byref(best)), lib.sslbm_set_tiles(other, None),
         lib.sslbm_set_tiles(other, ctypes.byref(Launch(4, 8, 0))),
         lib.sslbm_set_tiles(other, ctypes.byref(Launch(8, 8, 2))),
         lib.sslbm_set_tiles(other, ctypes.byref(Launch(99, 8, 1)))]
assert lib.sslbm_get_tiles(other) == 0
from paper_2603_19789_amd import Solver
s = Solver(300, 200, params(), dtype="f32")
assert "tiles" not in s.launch()
s.set_launch(4, 8, 1, tiles=True)
t = Solver(300, 200, params(), dtype="f32")
t.set_launch(**s.launch())
py = [s.launch(), t.launch(), t.plan(1000)["longest"]]
t.set_launch(4, 8, 1)
py_march = [t.launch(), t.plan(1000)["longest"]]
result = [a, b, march, codes, py, py_march]
''')
    assert a == b and {k[0] for k in a} == {"tile"} and {k[0] for k in march} == {"march"}
    assert codes == [-3, -1, -1, -3, -1]
    want = {"steps_per_pass": 4, "rows_per_wave": 8, "cols_per_lane": 1}
    assert py[0] == py[1] == {**want, "tiles": True} and py[2] > 4
    assert py_march == [want, 4]


def test_depth_with_a_diffusing_dead_compartment():
    """FP64 runs with a diffusing D: four steps a pass while two states fit the
    last-level cache, five beyond; without it, and in FP32, any size the same."""
    result = record('''
result = []
for n, d in ((1500, 3e-3), (1700, 3e-3), (1800, 3e-3), (2048, 3e-3), (4096, 3e-3), (1500, 0.0),
             (4096, 0.0)):
    result.append([passes(lambda: lib.sslbm_run(context(n, n, t, d), rho, scratch, 60, None))[0][1]
                   for t in ("f64", "f32")])
''')
    assert result == [[4, 6], [4, 6], [5, 6], [5, 6], [5, 6], [5, 6], [5, 6]]


def test_five_steps_where_they_save_passes():
    """FP64 with a diffusing D, four steps a pass on grids that the last-level
    cache holds: five where a run's passes take less time so."""
    result = record('''
result = []
for steps in (4, 5, 8, 9, 10, 12, 16, 17, 18, 19, 60):
    h = context(1024, 1024, "f64", 3e-3)
    ks = [k[1] for k in passes(lambda: lib.sslbm_run(h, rho, scratch, steps, None))]
    n, hi, lo = ctypes.c_longlong(), ctypes.c_int(), ctypes.c_int()
    lib.sslbm_plan_run(h, steps, ctypes.byref(n), ctypes.byref(hi), ctypes.byref(lo))
    assert [n.value, hi.value, lo.value] == [len(ks), max(ks), min(ks)]
    assert lib.sslbm_set_blocking(h, 4) == 0
    assert max(k[1] for k in passes(lambda: lib.sslbm_run(h, rho, scratch, steps, None))) <= 4
    result.append([steps, len(ks), max(ks)])
''')
    assert result == [[4, 2, 2], [5, 2, 3], [8, 2, 4], [9, 2, 5], [10, 2, 5], [12, 4, 3], [16, 4, 4],
                      [17, 4, 5], [18, 4, 5], [19, 6, 4], [60, 16, 4]]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_finite_difference_tiles_fit_low_grids(dtype):
    """The finite-difference step takes low tiles on grids of a few rows,
    however wide they are (columns, rows -> output rows of a tile)."""
    cases = [(65536, 1, 4), (262144, 4, 4), (65536, 5, 8), (65536, 16, 8), (65536, 17, 32),
             (200, 200, 4), (400, 400, 8), (2048, 2048, 32)]
    result = record(f'''
result = []
for nx, ny, _ in {cases!r}:
    h = context(nx, ny, {dtype!r})
    size = lib.sslbm_fd4_workspace_bytes(h)
    kinds = passes(lambda: lib.sslbm_fd4_run(h, rho, scratch, size, 3, None))
    (kernel, args, grid, *_), *rest = launched()
    rows = int(args[1]) * int(args[2]) - 16
    assert len(rest) == 2 and grid == -(-nx // 48) * -(-ny // rows)
    result.append([nx, ny, rows])
''')
    assert result == [list(c) for c in cases]


def test_bgk_depth_over_forms_of_grids():
    """Passes of several steps need rows and columns that are not mostly halo."""
    cases = [(150000, 1, 1, 1), (1000000, 1, 1, 1), (300000, 2, 5, 3), (31, 60000, 1, 1),
             (32, 60000, 7, 3), (256, 256, 1, 1), (1024, 1024, 5, 3), (2048, 2048, 7, 3)]
    result = record(f'''
result = []
for nx, ny, *_ in {cases!r}:
    row = [nx, ny]
    for dtype in ("f32", "f64"):
        h, d, ds = context(nx, ny, dtype), ctypes.c_void_p(4 << 40), ctypes.c_void_p(5 << 40)
        kinds = passes(lambda: lib.bgk_run(h, rho, d, scratch, ds, 210, None))
        row.append(max(k[1] for k in kinds))
    result.append(row)
''')
    assert result == [list(c) for c in cases]


def test_reported_bgk_plan_is_the_run_s():
    """BGK.plan, which the benchmark reports passes and traffic by, against the
    passes that are launched."""
    result = record('''
from paper_2603_19789_amd import BGK
result = []
for nx, ny in ((64, 64), (400, 400), (1100, 900), (4096, 4096), (200000, 1)):
    for dtype in ("f32", "f64"):
        b, d, ds = BGK(nx, ny, params(), dtype), ctypes.c_void_p(4 << 40), ctypes.c_void_p(5 << 40)
        for steps in (0, 1, 2, 7, 20, 63):
            kinds = passes(lambda: lib.bgk_run(b.handle, rho, d, scratch, ds, steps, None))
            took = [k[1] for k in kinds if k[0] == "bgk"]
            p = b.plan(steps)
            result.append([[len(took), max(took, default=0), min(took, default=0)],
                           [p["passes"], p["longest"], p["shortest"]]])
n = ctypes.c_longlong()
h, mobile = context(64, 64), context(64, 64, d_dead=1e-3)
result.append([[lib.bgk_plan_run(h, -1, ctypes.byref(n), None, None),
                lib.bgk_plan_run(h, 1, None, None, None),
                lib.bgk_plan_run(None, 1, ctypes.byref(n), None, None),
                lib.bgk_plan_run(mobile, 1, ctypes.byref(n), None, None)], [-1, -1, -1, -3]])
''')
    assert all(a == b for a, b in result), result


def test_rows_of_small_ensembles():
    """Automatic rows per wavefront of ensembles just too large for tiles: the
    faster of one and two wavefronts a SIMD, not a fixed least height."""
    cases = [(8, 512, 12), (6, 512, 16), (3, 1024, 14), (40, 512, 52)]
    result = record(f'''
result = []
for n, side, _ in {cases!r}:
    e = ensemble([(side, side)] * n)
    assert passes(lambda: lib.sslbm_ensemble_run(e, rho, scratch, 12, 0, None))
    info = binding.EnsembleClass()
    assert lib.sslbm_ensemble_class_info(e, 0, ctypes.byref(info)) == 0
    result.append([n, side, info.as_dict()["launch"]["rows_per_wave"]])
''')
    assert result == [list(c) for c in cases]


# (sizes and counts, kernels' columns a lane, chains): one chain at one column
# where the classes of odd rows hold most cells, where passes are short or where
# two columns cover more; else a chain of the even classes at two
MIXED = [([(1024, 1024, 14), (511, 511, 57)], [1, 2]), ([(1024, 1024, 16), (333, 333, 4)], [1, 2]),
         ([(2048, 2048, 4), (511, 300, 1), (200, 100, 3)], [1, 2]),
         ([(1024, 1024, 7), (1025, 1025, 40)], [1]), ([(400, 400, 30), (201, 201, 30)], [1]),
         ([(256, 256, 412), (301, 301, 33)], [1]), ([(1024, 1024, 20), (512, 512, 20)], [2]),
         ([(1025, 1025, 20), (511, 512, 20)], [1])]


def test_columns_of_ensembles_with_odd_rows():
    """Classes of even rows keep two columns a lane beside odd ones on large
    ensembles; a class that runs alone takes the columns of its own sizes."""
    result = record(f'''
result = []
for groups, want in {MIXED!r}:
    sizes = [(nx, ny) for nx, ny, n in groups for _ in range(n)]
    e = ensemble(sizes)
    passes(lambda: lib.sslbm_ensemble_run(e, rho, scratch, 12, 0, None))
    ks = [l for l in launched() if l[0] == "ensemble_march_kernel"]
    alone = []
    for c in range(lib.sslbm_ensemble_class_count(e)):
        passes(lambda: lib.sslbm_ensemble_run_class(e, c, rho, scratch, 12, None))
        alone += [int(l[1][3]) for l in launched() if l[0] == "ensemble_march_kernel"][:1]
    double = ensemble(sizes, "f64")
    passes(lambda: lib.sslbm_ensemble_run(double, rho, scratch, 20, 0, None))
    f64 = [l for l in launched() if l[0] == "ensemble_march_kernel"]
    result.append([want, sorted({{int(l[1][3]) for l in ks}}), len(ks), alone, len(f64)])
''')
    for want, cols, count, alone, f64 in result:
        assert cols == want and count == 2 * len(want) and f64 == 4, (want, cols, count, f64)
    assert result[0][3] == [1, 2] and result[3][3] == [2, 1]  # by class, in order of size


def test_model_runs_of_one_pass():
    """A generic model's run that one pass can take: one pass and a copy on
    large grids, two passes where the last-level cache holds the states."""
    result = record('''
from paper_2603_19789_amd import Model
result = []
for dtype, n, steps in (("f32", 1024, 2), ("f32", 2600, 2), ("f32", 2600, 3), ("f32", 4096, 3),
                        ("f64", 1600, 2), ("f64", 2048, 2), ("f64", 2048, 3), ("f64", 4096, 3),
                        ("f32", 4096, 1), ("f32", 4096, 4), ("f32", 4096, 6), ("f32", 4096, 7)):
    m = Model(n, n, inputs.seirvd_model(lattice=5), dtype=dtype)
    kinds = [k[0] for k in passes(lambda: lib.sslbm_model_run(m.handle, rho, scratch, steps, None))]
    result.append([dtype, n, steps, len(kinds) - kinds.count("copy"), kinds.count("copy")])
''')
    want = {("f32", 1024, 2): (2, 0), ("f32", 2600, 2): (1, 1), ("f32", 2600, 3): (2, 0),
            ("f32", 4096, 3): (1, 1), ("f64", 1600, 2): (2, 0), ("f64", 2048, 2): (1, 1),
            ("f64", 2048, 3): (2, 0), ("f64", 4096, 3): (1, 1), ("f32", 4096, 1): (1, 1),
            ("f32", 4096, 4): (2, 0), ("f32", 4096, 6): (2, 0), ("f32", 4096, 7): (4, 0)}
    assert {tuple(r[:3]): tuple(r[3:]) for r in result} == want


def test_an_ensemble_run_is_planned_once():
    """A run that repeats the last one's steps makes no new plan; one with other
    steps, or after a change of shapes, does."""
    first, again, changed, shapes = record('''
e = ensemble([(65 + 7 * i, 90 + 3 * i) for i in range(20)] + [(300, 200)])
run = lambda n: passes(lambda: lib.sslbm_ensemble_run(e, rho, scratch, n, 0, None))
a = run(6); first = rec.rec_queries()
b = run(6); again = rec.rec_queries()
assert a == b and {k[0] for k in a} == {"tile"}
run(60); changed = rec.rec_queries()
assert lib.sslbm_ensemble_set_launch(e, ctypes.byref(Launch(3, 16, 1))) == 0
c = run(60)
assert lib.sslbm_ensemble_set_launch(e, ctypes.byref(Launch(0, 0, 0))) == 0
d = run(60)
result = [first, again, changed, [len(c), sorted({k[0] for k in c}), sorted({k[0] for k in d})]]
''')
    assert again == 1 < min(first, changed)  # one query: the device the ensemble is on
    assert shapes == [20, ["ensemble_march_kernel"], ["tile"]]


@pytest.mark.parametrize("dtype", ["f32", "f64"])
def test_launches_without_an_answer_from_the_device(dtype):
    """Where the device cannot be asked for its compute units the launchers
    take an MI355X's, and the query's error is not the launches' one."""
    result = record(f'''
calls = []
for there in (1, 0):
    h, d, ds = context(1024, 900, {dtype!r}), ctypes.c_void_p(4 << 40), ctypes.c_void_p(5 << 40)
    size = lib.sslbm_fd4_workspace_bytes(h)
    rec.rec_device(there)
    row = []
    for call in (lambda: lib.bgk_run(h, rho, d, scratch, ds, 30, None),
                 lambda: lib.sslbm_fd4_run(h, rho, scratch, size, 4, None),
                 lambda: lib.sslbm_run(h, rho, scratch, 30, None)):
        rec.rec_clear()
        row.append([call(), [l[:3] for l in launched()]])
    calls.append(row)
result = calls
''')
    asked, unasked = result
    assert [c[0] for c in asked + unasked] == 6 * [0]
    assert unasked[:2] == asked[:2] and unasked[2][1]


@pytest.mark.parametrize("d_dead", [0.0, 3e-3])
def test_compared_sizes_take_every_tile_height(d_dead):
    """The sizes whose tiles the GPU tests compare with the march cover every
    tile height there is, on single grids and in ensembles."""
    from test_gpu_ensemble_tiles import HEIGHTS
    single, many = record(f'''
single = {{}}
for dtype in ("f32", "f64"):
    rows = set()
    for nx, ny, steps in {_tile_shapes()!r}:
        h = context(nx, ny, dtype, {d_dead})
        rows |= {{k[2] for k in passes(lambda: lib.sslbm_run(h, rho, scratch, steps, None))
                 if k[0] == "tile"}}
    single[dtype] = sorted(rows)
many = []
for dtype, rows, steps, sizes in {HEIGHTS!r}:
    e = ensemble(sizes, dtype, {d_dead})
    kinds = passes(lambda: lib.sslbm_ensemble_run(e, rho, scratch, steps, 0, None))
    many.append([dtype, *sorted({{k[2] for k in kinds if k[0] == "tile"}})])
result = [single, many]
''')
    assert single == {"f32": [2, 3, 4, 5, 7], "f64": [1, 2, 3]}
    assert many == [[dtype, rows] for dtype, rows, *_ in HEIGHTS]


def _tile_shapes():
    from test_gpu_tiles import SHAPES
    return SHAPES
