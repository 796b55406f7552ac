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
