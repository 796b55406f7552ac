"""Plans of the uneven batch on the host (fake_hip.py): what they allocate, what
they do where that fails, and which kernels their calls take."""
import pytest

from fake_hip import script


def test_default_routes(tmp_path_factory):
    got = script("""
rc, p = plan([(HEX, 300, 16384, 65536)])
rc2, q = plan([(HEX, 300, 16384, 65536)], flags=_lib.PSDF_BATCH_EXHAUSTIVE)
rc3, s = plan([(HEX, 300, 1000, 4000)])
emit([rc, rc2, rc3, run(p), bound(p), run(q)[0], run(s)[0]])
""", tmp_path_factory)
    assert got == [0, 0, 0, ["cull_list", "cull_stage_kernel"], ["cull_list", "cull_stage_kernel"],
                   "batch_kernel", "batch_kernel"]


def test_no_room_for_the_culled_tables(tmp_path_factory):
    """A plan that has room for the full evaluation alone takes it: whichever of
    the culled tables does not fit, and with a limit between the two sizes."""
    got = script("""
insts = [(HEX, 300, 16384, 65536)]
rc, q = plan(insts, flags=_lib.PSDF_BATCH_EXHAUSTIVE)
full = hip.fake_used()
lib.psdf_batch_plan_destroy(q)
rc, p = plan(insts)
culled = hip.fake_used()
lib.psdf_batch_plan_destroy(p)
out = []
for limit in (full, full + 65536, culled - 1, culled):
    hip.fake_limit(limit)
    rc, p = plan(insts)
    out.append([rc, run(p)[0] if rc == 0 else None, hip.fake_used() in (full, culled)])
    lib.psdf_batch_plan_destroy(p)
    out[-1].append(hip.fake_used())
hip.fake_limit(full - 1)
rc, p = plan(insts)
out.append([rc, hip.fake_used()])
hip.hipGetLastError()
hip.fake_limit(2**63)
for k in range(40):
    hip.fake_fail_malloc(k)
    rc, p = plan(insts)
    if rc == 0:
        out.append([run(p)[0], hip.fake_used() in (full, culled)])
        lib.psdf_batch_plan_destroy(p)
    hip.hipGetLastError()
    assert hip.fake_used() == 0, k
emit(out)
""", tmp_path_factory)
    fallback = [0, "batch_kernel", True, 0]
    assert got[:4] == [fallback, fallback, fallback, [0, "cull_list", True, 0]]
    assert got[4] == [-6, 0]
    rest = got[5:]
    assert rest.count(["batch_kernel", True]) == 5          # the five culled tables
    assert rest.count(["batch_kernel", True]) + rest.count(["cull_list", True]) == len(rest)


def test_no_room_for_the_staged_boxes(tmp_path_factory):
    """Staging takes the circles and rows, as it did, where the boxes and records
    of the culled form do not fit; the bound form then reads the edges."""
    got = script("""
insts = [(HEX, 300, 16384, 65536)]
out = []
rc, p = plan(insts)
before = hip.fake_used()
rows = 16384 * (16 + 40 * 4 + 16)
for limit in (before + rows, before + rows + 16 * 16384, before + rows + 80 * 16384):
    hip.fake_limit(limit)
    out.append([*stage(p), hip.fake_used() - before, bound(p), run(p)])
lib.psdf_batch_plan_destroy(p)
emit([out, hip.fake_used()])
""", tmp_path_factory)
    rows, both = 16384 * 192, ["cull_list", "cull_stage_kernel"]
    assert got[1] == 0
    assert got[0] == [[0, ["stage_batch"], rows, both, both], [0, ["stage_batch"], rows, both, both],
                      [0, ["stage_batch", "cull_stage_edges"], rows + 80 * 16384, both, both]]


NEEDLE = "[[-0.5, 0.0], [0.5, -2e-6], [0.5, 2e-6]]"


def test_tuning_decides_for_its_own_plan(tmp_path_factory):
    """What autotuning found, the culled or the full evaluation, holds for the
    plan that was tuned: the choice depends on the map and the footprints, which
    the cache's size signature does not know.  (On this runtime the form of fewer
    launches is the faster: the full one for one footprint size, where they are
    equal, the culled one for two.)"""
    got = script("""
one = [(HEX, 300, 16384, 65536)]
two = [(HEX, 300, 16384, 65536), (HEX[::2], 300, 16384, 65536)]
T, X = _lib.PSDF_BATCH_AUTOTUNE, _lib.PSDF_BATCH_EXHAUSTIVE
out = []
for insts in (one, two):
    rc, p = plan(insts, flags=T)
    autotune(p)
    rc, later = plan(insts)
    out.append([run(p)[0], run(later)[0]])
    rc, x = plan(insts, flags=T | X)
    autotune(x)
    rc, later = plan(insts)
    out.append([run(x)[0], run(later)[0]])
emit(out)
""", tmp_path_factory)
    assert got == [["batch_kernel", "cull_list"], ["batch_kernel", "cull_list"],
                   ["cull_list", "cull_list"], ["batch_kernel", "cull_list"]]


def test_cache_files(tmp_path_factory, tmp_path):
    """Lines of a cache file give a shape and never the form, also those written
    with the form in their last number; a footprint without a bound is not culled."""
    path = tmp_path / "tune"
    got = script(f"""
insts = [(HEX, 300, 16384, 65536)]
rc, p = plan(insts, flags=_lib.PSDF_BATCH_AUTOTUNE)
autotune(p)
line = open({str(path)!r}).read().split()
emit(line)
""", tmp_path_factory, env={"PSDF_TUNE_CACHE": str(path)})
    assert len(got) == 4 and got[3] in ("0", "1")
    sig = got[0]
    for last in range(6):
        path.write_text(f"{sig} 8 4 {last}\n")
        got = script(f"""
info = [ctypes.c_int32() for _ in range(5)]
rc, p = plan([(HEX, 300, 16384, 65536)])
lib.psdf_batch_plan_info(p, *[ctypes.byref(i) for i in info])
rc, q = plan([({NEEDLE}, 300, 16384, 65536)])
emit([run(p)[0], run(q)[0], info[0].value, info[1].value, info[4].value])
""", tmp_path_factory, env={"PSDF_TUNE_CACHE": str(path)})
        assert got == ["cull_list", "batch_kernel", 8, 256, last & 1], last


def test_bound_form_follows_the_plan(tmp_path_factory):
    """psdf_batch_screened_bound is culled where psdf_batch is: not after an
    explicit shape, nor where tuning found the full evaluation faster."""
    got = script("""
one = [(HEX, 300, 16384, 65536)]
out = []
rc, p = plan(one)
out.append([bound(p), stage(p)[1]])
lib.psdf_batch_set_shape(p, 8, 64, 1)
out.append([run(p)[0], "screen_bound" in bound(p), stage(p)[1]])
rc, p = plan(one, flags=_lib.PSDF_BATCH_AUTOTUNE)
stage(p)
autotune(p)
out.append([run(p)[0], "screen_bound" in bound(p), stage(p)[1]])
emit(out)
""", tmp_path_factory)
    both = ["cull_list", "cull_stage_kernel"]
    assert got == [[both, ["stage_batch", "cull_stage_edges"]],
                   ["batch_kernel", True, ["stage_batch"]], ["batch_kernel", True, ["stage_batch"]]]


def test_eps_that_leaves_edges_without_a_bound(tmp_path_factory):
    """An edge shorter than 4e6 eps leaves its obstacle without a bound: beyond a
    centimetre, where ordinary maps have such edges, calls take the full evaluation."""
    got = script("""
out = []
for eps in (1e-12, 2e-9, 3e-9, 1e-7, 1e-3):
    par = params(eps=eps)
    rc, p = plan([(HEX, 300, 16384, 65536)], par=par)
    out.append([run(p)[0], bound(p)[0] == "cull_list", plain(HEX, 50, 65536, par=par)[0]])
emit(out)
""", tmp_path_factory)
    culled, full = ["cull_list", True, "cull_main"], ["batch_kernel", False, "main_kernel"]
    assert got == [culled, culled, full, full, full]


def test_bound_form_where_eps_leaves_no_bound(tmp_path_factory):
    """Where eps moves the evaluation's distances by more than the circles have to
    spare, the bound form evaluates every pair, as psdf_batch does; below, plans
    that are not culled for their eps are screened by circles, as they were."""
    got = script("""
out = []
for insts in ([(HEX, 300, 16384, 65536)], [(HEX, 20, 100, 400)]):
    for eps in (3e-9, 1e-6, 2e-6, 1e-2):
        rc, p = plan(insts, par=params(eps=eps))
        out.append(["screen_bound" in bound(p), run(p)])
        out[-1].append(bound(p) == out[-1][1])
        assert stage(p)[0] == 0
        out[-1].append(bound(p) == out[-1][1])
        del out[-1][1]
emit(out)
""", tmp_path_factory)
    assert got == 2 * [[True, False, False], [True, False, False],
                       [False, True, True], [False, True, True]]


def test_sizes_and_footprints_that_are_culled(tmp_path_factory):
    """Small maps, and footprints with a sharp corner, against which what is no
    convex polygon has a loose bound, ask for larger problems."""
    got = script("""
def needle(w):
    return [[-0.5, 0.0], [0.5, -w], [0.5, w]]
blunt, thin, thinner = needle(0.176), needle(0.0437), needle(8.7e-4)
batches = [run(plan([(fp, N, M, 4 * M)] * k)[1])[0] == "cull_list" for fp, k, N, M in (
    (blunt, 1, 300, 16384), (thin, 1, 300, 16384), (thin, 1, 2000, 16384), (thin, 16, 64, 16384),
    (thinner, 16, 64, 16384), (thinner, 1, 2000, 16384), (thinner, 1, 20000, 2048))]
calls = [plain(fp, N, M, mbar=b)[0] == "cull_main" for fp, N, M, b in (
    (blunt, 100, 16384, 4), (thin, 100, 16384, 4), (thin, 200, 16384, 4), (thinner, 200, 16384, 4),
    (thinner, 600, 16384, 4), (HEX, 20000, 64, 8), (HEX, 20000, 65, 8), (HEX, 20000, 64, 16),
    (HEX[:3], 20000, 320, 4), (HEX[:3], 20000, 321, 4), (HEX[:3], 20000, 128, 8), (HEX[:3], 20000, 129, 8))]
emit([batches, calls])
""", tmp_path_factory)
    assert got == [[True, False, True, True, False, True, True],
                   [True, False, True, False, True, False, True, True, False, True, False, True]]


def test_routes_of_the_needle_tests(tmp_path_factory):
    """The sizes of test_gpu_cull_needles.py are culled."""
    got = script("""
def needle(w):
    return [[-0.5, 0.0], [0.5, -w], [0.5, w]]
out = []
for w in (0.1, 0.0437, 8.7e-4, 2e-6):
    rc, p = plan([(HEX, 300, 16384, 65536)] + [(needle(w), N, M, 4 * M) for N, M in ((30, 1000), (70, 908), (3, 18))])
    out.append(run(p)[0])
for w in (0.1, 0.0437, 8.7e-4):
    out.append(plain(needle(w), 300, 30011)[0])
emit(out)
""", tmp_path_factory)
    assert got == 4 * ["cull_list"] + 3 * ["cull_main"]


def test_batches_that_read_an_obstacle_for_few_stages(tmp_path_factory):
    """Instances of more than 64 segments, and wide obstacles, ask for more stages; the
    sizes of test_gpu_cull_long.py are culled."""
    got = script("""
def route(k, N, M, mbar):
    rc, p = plan([(HEX, N, M, M * mbar)] * k, mbar=mbar)
    r = run(p)[0]
    lib.psdf_batch_plan_destroy(p)
    return r == "cull_list"
few = [route(*c) for c in ((20, 1, 210000, 4), (3, 16, 130000, 4), (1, 120, 130000, 4), (70, 1, 60000, 4),
                           (257, 1, 16384, 8), (257, 2, 16384, 8), (65, 5, 16384, 16), (65, 6, 16384, 16),
                           (3, 12, 130000, 8), (2, 32, 130000, 8), (3, 16, 130000, 16))]
long = [route(1, 150, 70000, mbar) for mbar in (4, 8, 16)]
for M in (65536, 65537, 140000):
    rc, p = plan([(HEX, 300, 16384, 65536)] + [(HEX[::2], N, M, 4 * M) for N in (70, 60, 1)])
    long.append(run(p)[0] == "cull_list")
emit([few, long])
""", tmp_path_factory)
    assert got == [[False, False, True, True, False, True, False, True, False, True, True], 6 * [True]]


def test_small_calls(tmp_path_factory):
    """A quad of lanes per obstacle for few stages; not for more than 32 free segments,
    whose one edge a quad evaluates four times."""
    got = script("""
emit([plain(HEX, N, M, mbar=b)[0] for N, M, b in (
    (50, 16, 1), (50, 32, 1), (50, 33, 1), (1, 128, 1), (50, 33, 2), (50, 128, 4), (300, 128, 4), (50, 129, 4))])
""", tmp_path_factory)
    quad, lane = "small_quad", "small_kernel"
    assert got == [quad, quad, lane, lane, quad, quad, lane, lane]


def test_soft_minimum_that_reaches_far(tmp_path_factory):
    """A stage looks at all obstacles within log(axes) / eta."""
    got = script("""
out = []
for par in (params(eta=1000.0), params(eta=1.0), params(eta=0.1), params(eta=float("inf")), params(eps_sat=1.0),
            params(eps_sat=20.0)):
    rc, p = plan([(HEX, 300, 16384, 65536)], par=par)
    out.append(run(p)[0] == "cull_list")
emit(out)
""", tmp_path_factory)
    assert got == [True, True, False, True, True, False]


def test_bound_form_of_plans_that_the_batch_does_not_cull(tmp_path_factory):
    """Where a footprint, the stages per obstacle or eta speak against it, psdf_batch is
    not culled; the bound form still is, and the tuner still times the culled form (here
    the form of fewer launches is the faster)."""
    got = script("""
def needle(w):
    return [[-0.5, 0.0], [0.5, -w], [0.5, w]]
out = []
for insts, mbar, par in (([(needle(8.7e-4), 300, 16384, 65536)], 4, None), ([(HEX, 2, 16384, 16384 * 16)] * 130, 16, None),
                         ([(HEX, 300, 16384, 65536)], 4, params(eta=0.1))):
    rc, p = plan(insts, mbar=mbar, par=par)
    out.append([run(p)[0], bound(p), stage(p)[1], bound(p)])
    lib.psdf_batch_set_shape(p, 8, 64, 1)
    out[-1].append("screen_bound" in bound(p))
    rc, p = plan(insts + [(HEX[:5], 1, 1, 1)], mbar=mbar, par=par, flags=_lib.PSDF_BATCH_AUTOTUNE)
    autotune(p)
    out[-1].append(run(p)[0])
emit(out)
""", tmp_path_factory)
    both = ["cull_list", "cull_stage_kernel"]
    want = ["batch_kernel", both, ["stage_batch", "cull_stage_edges"], both, True, "cull_list"]
    assert got == 3 * [want]
