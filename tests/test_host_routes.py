"""Which way a call goes -- what it allocates and launches, what it refuses -- read from the host code on a machine
without a GPU (fake_hip.py)."""
import os
import re

import pytest

import paper_2512_02551_amd as hg
from fake_hip import ask

CSRC = os.path.join(os.path.dirname(os.path.abspath(hg.__file__)), "csrc")


def table_rows(tn):
    text = open(os.path.join(CSRC, "dispatch_table_tn.inc" if tn else "dispatch_table.inc")).read()
    rows = [(tuple(int(v) for v in m[:3]), m[3]) for m in re.findall(r'\{\s*(\d+),\s*(\d+),\s*(\d+),\s*"([^"]*)"', text)]
    rows = [r for r in rows if min(r[0]) > 0 and r[1]]
    assert len(rows) > 1000
    return rows


@pytest.mark.parametrize("tn", [False, True])
def test_the_static_entry_point_runs_every_table_row_whose_workspace_fits(tn):
    """A workspace of up to HGEMM_STATIC_SCRATCH_BYTES, that size included: the launches of the planned call."""
    shapes = [s for s, _ in table_rows(tn)]
    full = 0
    for (m, n, k), r in zip(shapes, ask([{"M": m, "N": n, "K": k, "tn": tn} for m, n, k in shapes])):
        assert r["plan"] == 0 and r["run"] == 0
        if r["workspace"] > hg.STATIC_SCRATCH_BYTES:
            continue
        full += r["workspace"] == hg.STATIC_SCRATCH_BYTES
        assert r["static"] == 0, (m, n, k, r["describe"], r["workspace"])
        assert r["static_log"] == r["run_log"], (m, n, k, r["describe"])
    assert full > 0


def kernels(log):
    """Names and grids of the launches of a log."""
    out = []
    for line in log:
        if line.startswith("launch "):
            name, x, y, *args = line.split()[1:]
            out.append((re.search(r"([a-z0-9_]+_kernel)", re.sub(r"^_ZN5hgemm\d+", "", name))[1], int(x), int(y), *map(int, args)))
    return out


@pytest.mark.parametrize("tn", [False, True])
@pytest.mark.parametrize("m,n,k", [(3, 1001, 1003), (2, 4099, 520), (266, 360, 280), (100, 1001, 1008)])
def test_a_pitch_of_c_beyond_32_bits_keeps_the_matrix_core_kernels(m, n, k, tn):
    """Rows of C 2^31 elements apart and more: stored packed and copied from there; one row: stored in place."""
    qs = [{"M": rows, "N": n, "K": k, "tn": tn, "ldc": (1 << 31) + pad} for rows in (m, 1) for pad in (3, 1 << 31)]
    qs.append({"M": m, "N": n, "K": k, "tn": tn, "ldc": (1 << 31) - 1})
    for q, r in zip(qs, ask(qs)):
        if q["M"] * n * k < 1 << 20:
            assert r["describe"] == "generic"
            continue
        names = [name for name, *_ in kernels(r["run_log"])]
        assert r["run"] == 0 and "generic_gemm_kernel" not in names, (q, names)
        assert ("copy_back_kernel" in names) == (q["M"] > 1 and q["ldc"] >= 1 << 31), (q, names)
        assert r["static"] == 0 and r["static_log"] == r["run_log"], q


MIB = 1 << 20


@pytest.mark.parametrize("q,needs", [
    ({"M": 16, "N": 50257, "K": 4096, "tn": True}, 0),                       # nothing is copied
    ({"M": 300, "N": 4097, "K": 4096, "tn": True, "lda": 4099}, 18 * MIB),   # A is (the rest: planes)
    ({"M": 2500, "N": 2504, "K": 2501}, 13 * MIB),                           # A is; B, of fewer rows than the copy of A has columns, is not
], ids=["none", "A", "A, short B"])
def test_no_memory_for_copies_that_no_aligned_call_needs(q, needs):
    """The room for copies of operands that can be read where they lie serves misaligned bases only: where the device has no
    memory for it, the plan keeps the matrix-core kernel, and a misaligned call takes the generic kernel on the caller's operands."""
    from fake_hip import BASE
    rich, poor, a_off, b_off, rich_off = ask([q, {**q, "memory": needs}, {**q, "memory": needs, "A": BASE + 2}, {**q, "memory": needs, "B": BASE + 2},
                                              {**q, "A": BASE + 2, "B": BASE + 2}])
    assert rich["workspace"] > needs and rich["describe"] == poor["describe"] and "generic" not in poor["describe"]
    assert poor["workspace"] <= needs and poor["run"] == 0 and poor["run_log"] == rich["run_log"]
    assert [k[0] for k in kernels(rich_off["run_log"])][0] == "pad_copy_kernel" and "generic_gemm_kernel" not in str(rich_off["run_log"])
    copies_a = "pad_copy_kernel" in str(rich["run_log"])
    for r, off in ((a_off, "A"), (b_off, "B")):
        last = kernels(r["run_log"])[-1]
        assert r["run"] == 0
        if off == "A" and copies_a:
            assert r["run_log"] == poor["run_log"]                 # its copy is made either way
            continue
        assert last[0] == "generic_gemm_kernel", r["run_log"]
        M, N, K, tn = q["M"], q["N"], q["K"], q.get("tn", False)
        up8 = (K + 7) // 8 * 8
        assert last[3:] == ((last[3] if copies_a else BASE + 2 * (off == "A")), BASE + 2 * (off == "B"), BASE, M, N, K,
                            up8 if copies_a else q.get("lda", K), K if tn else N, N), last


def test_no_memory_for_the_planes_of_a_phased_split():
    """... and the same tile runs without a split."""
    rich, poor = ask([{"M": 512, "N": 8192, "K": 16384}, {"M": 512, "N": 8192, "K": 16384, "memory": 32 * MIB}])
    assert "sk=4" in rich["describe"] and "ph=1" in rich["describe"] and rich["workspace"] == 64 * MIB
    assert poor["describe"] == rich["describe"].replace("sk=4", "sk=1") and poor["workspace"] == 0 and poor["run"] == 0


@pytest.mark.parametrize("tn", [False, True])
def test_no_phased_table_row_has_less_than_two_k_tiles(tn):
    """The phased schedule copies two K-tiles ahead: with one (12288 x 16384 x 64), half of its copies move zeros and it is 28-35 % slower."""
    phased = [(shape, spec) for shape, spec in table_rows(tn) if "ph=1" in spec]
    assert len(phased) > 200
    for (m, n, k), spec in phased:
        assert k // int(re.search(r"sk=(\d+)", spec)[1]) >= 128, (m, n, k, spec)


@pytest.mark.parametrize("m,n,k,streamed", [(62, 473671, 48, False), (33, 80001, 255, False), (33, 80001, 256, True), (64, 8001, 2048, False),
                                            (32, 80001, 255, True), (32, 4001, 300, True)])
def test_which_unaligned_row_major_b_is_streamed_where_it_lies(m, n, k, streamed):
    """Up to 32 rows of A always, up to 64 from 32 MiB of B and K = 256 on; the others are copied."""
    (r,) = ask([{"M": m, "N": n, "K": k}])
    reads_any_b = "skinny_gemm_kernel" in str(r["run_log"]) and any("skinny_gemm_kernel" in line and "ELb1EEEvNS_8GemmArgsE" in line for line in r["run_log"])
    assert r["run"] == 0 and reads_any_b == streamed, r["run_log"]


def test_in_place_off_the_grid_takes_no_split_across_the_allocation_step():
    """hipMalloc costs 60 us more from 2 MiB on, which a program that plans on every call pays: where the copies stay below, so do the planes."""
    shapes = [(411, 279, 1277, False), (125, 198, 980, False), (295, 143, 1052, True), (380, 301, 1301, True), (640, 163, 1601, False), (250, 417, 1201, True)]
    for (m, n, k, tn), r in zip(shapes, ask([{"M": m, "N": n, "K": k, "tn": tn} for m, n, k, tn in shapes])):
        copies = 2 * (m * (k + 7) + (n + 7) * (k + 7))
        assert r["run"] == 0 and (r["workspace"] < 2 * MIB or copies > 2 * MIB - 65536), (m, n, k, r["describe"], r["workspace"])


def batch_sets(n, m, nn, k, lda=0):
    """n sets of packed operands (rows of A lda apart), one behind the other with nothing between them."""
    from fake_hip import BASE
    a, b, c = 2 * m * (lda or k), 2 * k * nn, 2 * m * nn
    return [(BASE + i * (a + b + c), BASE + i * (a + b + c) + a, BASE + i * (a + b + c) + a + b) for i in range(n)]


def many(sets, m=256, n=256, k=256, **more):
    (r,) = ask([{"M": m, "N": n, "K": k, "many": sets, **more}])
    return r["many"], [int(line.split()[2]) if "BatchArgs" in line else 1 for line in r["many_log"] if line.startswith("launch ")]


def test_small_calls_of_a_batch_share_launches_where_none_depends_on_another():
    """Problems per launch of hgemm_run_many.  Calls join a launch as long as no call of it writes what another reads or writes."""
    s = batch_sets(8, 256, 256, 256)
    assert many(s) == (0, [8])
    assert many(batch_sets(70, 256, 256, 256)) == (0, [32, 32, 6])
    assert many(batch_sets(33, 256, 256, 256)) == (0, [32, 1])
    assert many(s, count=19, first=3) == (0, [8, 8, 3])                               # a set's C comes round again
    assert many(s[:1], count=4) == (0, [1] * 4)
    chain = [(s[0][0], s[0][1], s[0][2]), (s[0][2], s[1][1], s[1][2]), (s[2][0], s[2][1], s[2][2]), (s[1][0], s[2][2], s[3][2])]
    assert many(chain) == (0, [1, 2, 1])                                              # A is the C of the call before; B is
    assert many([s[0], (s[1][0], s[0][1], s[1][2]), (s[1][0], s[0][1], s[2][2])]) == (0, [3])     # operands that are only read may be shared
    assert many([s[0], (s[1][0], s[1][1], s[0][0]), s[2]]) == (0, [1, 2])             # C is an A of the call before
    assert many([s[0], (s[1][0], s[1][1], s[0][2] + 2 * 256 * 255 + 2 * 248), s[2]]) == (0, [1, 2])   # the last 16 bytes of its C
    assert many([s[0], (s[1][0], s[1][1] + 2, s[1][2]), s[2], s[3]]) == (0, [1, 1, 2])            # a misaligned B goes its own way
    status, launches = many([s[0], s[1], (s[2][0], None, s[2][2]), s[3]])
    assert status != 0 and launches == [2]                                            # calls in front of the one that fails are enqueued


def test_the_tiles_of_a_shared_launch_follow_from_the_calls_it_holds():
    """500 x 512 x 520 has 16 tiles of 128 x 128 and 64 of 64 x 64: the wide ones where the launch's own calls give each of 256 compute units
    one, not where a later launch of the batch holds fewer calls, or calls that depend on each other cut it short."""
    def launches(sets):
        (r,) = ask([{"M": 500, "N": 512, "K": 520, "many": sets}])
        assert r["many"] == 0
        return [(x, y) for _, x, y, *_ in kernels(r["many_log"])]

    s = batch_sets(40, 500, 512, 520)
    assert launches(s) == [(32, 16), (8, 64)]
    assert launches(s[:16]) == [(16, 16)] and launches(s[:15]) == [(15, 64)]
    assert launches(batch_sets(34, 500, 512, 520)) == [(32, 16), (2, 64)]
    pairs = [(a, b, s[i // 2 % 2][2]) if i % 2 else (a, b, c) for i, (a, b, c) in enumerate(s[2:22])]      # two places for C come round in every second call
    assert [x for x, y in launches(pairs)] == [5, 4, 4, 4, 3] and {y for _, y in launches(pairs)} == {64}


def test_bench_times_the_kernel_that_its_row_names():
    """A row over rotating operand sets runs the planned kernel once a call, not shared launches of another one."""
    import bench

    class FakePlan:
        def __init__(self, m, n, k, layouts, spec):
            (self.r,) = ask([{"M": m, "N": n, "K": k, "many": batch_sets(6, m, n, k), **({"spec": spec} if spec else {})}])
            assert self.r["plan"] == 0

        def describe(self):
            return self.r["describe"]

        def destroy(self):
            pass

    class Library:
        Plan = FakePlan

    for shape in ((512, 512, 512), (64, 512, 256), (200, 201, 203)):
        planned = FakePlan(*shape, None, None)
        timed = bench.plan_to_time(Library, shape, None, None, 6)
        assert timed.describe() == planned.describe()
        assert timed.r["many_log"] == 6 * planned.r["run_log"], timed.r["many_log"]
        assert bench.plan_to_time(Library, shape, None, None, 1).r["run_log"] == planned.r["run_log"]


def test_which_plans_share_launches():
    """Small unsplit problems in both layouts and in wider buffers; not large ones, split ones or those off the 16-byte grid."""
    assert many(batch_sets(4, 16, 64, 64), 16, 64, 64, tn=True) == (0, [4])
    assert many(batch_sets(5, 100, 200, 304, lda=512), 100, 200, 304, lda=512) == (0, [5])
    assert many(batch_sets(3, 1536, 1536, 1536), 1536, 1536, 1536) == (0, [1] * 3)
    assert sum(many(batch_sets(3, 64, 64, 16384), 64, 64, 16384)[1]) >= 3             # split: two launches or fused, one call each
    assert max(many(batch_sets(3, 64, 64, 16384), 64, 64, 16384)[1]) == 1
    assert max(many(batch_sets(3, 200, 201, 203), 200, 201, 203)[1]) == 1


@pytest.mark.parametrize("m,n,k,tn,launches", [(1000, 1001, 1003, False, 1), (500, 501, 503, True, 1), (70, 3001, 1001, False, 1), (264, 328, 200, False, 1), (90, 71, 4101, False, 2),
                                               (700, 71, 3301, True, 2)])
def test_small_problems_off_the_grid_are_read_where_they_lie(m, n, k, tn, launches):
    """No copies: one launch (a split in planes: two), no workspace but for planes, whatever the bases; the static entry point launches the same."""
    from fake_hip import BASE
    pads = {"lda": k + 1, "ldb": (k if tn else n) + 3} if (m, n, k) == (264, 328, 200) else {}
    plain, off = ask([{"M": m, "N": n, "K": k, "tn": tn, **pads}, {"M": m, "N": n, "K": k, "tn": tn, "A": BASE + 2, "B": BASE + 6, "C": BASE + 2, **pads}])
    names = [name for name, *_ in kernels(plain["run_log"])]
    assert ",di=1" in plain["describe"] and plain["describe"].endswith("pad=1") and len(names) == launches and names[0] == "mfma_gemm_kernel", plain
    assert "sk=1," in plain["describe"] and plain["workspace"] == 0 or "sk=1," not in plain["describe"] and plain["workspace"] > 0
    assert off["run_log"] == plain["run_log"] and plain["static"] == 0 and plain["static_log"] == plain["run_log"]


def test_what_the_static_entry_point_refuses_stays_refused():
    """Problems whose padded copies exceed the scratch are refused, also where the kernels that read them in place would need none."""
    thin = {"M": 40, "N": 190001, "K": 201, "tn": True}
    (r,) = ask([thin])
    assert r["plan"] == 0 and r["static"] == 6, r


@pytest.mark.parametrize("m,n,k,tn", [(4100, 4101, 4103, False), (2216, 1408, 419, False), (3463, 79, 5896, True), (16, 50257, 4096, False), (16, 50257, 4096, True)])
def test_problems_off_the_grid_that_keep_their_copies_streams_and_phased_kernels(m, n, k, tn):
    (r,) = ask([{"M": m, "N": n, "K": k, "tn": tn}])
    assert r["run"] == 0 and ",di=1" not in r["describe"], r


@pytest.mark.parametrize("q,in_place", [
    ({"M": 1980, "N": 13416, "K": 104, "tn": True, "lda": 124}, False), ({"M": 3992, "N": 1311, "K": 71, "tn": True}, False),     # storing C is most of it
    ({"M": 2801, "N": 1427, "K": 71}, True), ({"M": 1720, "N": 2342, "K": 243}, True),                                          # up to 4M elements; four K-tiles
    ({"M": 53, "N": 53440, "K": 3213}, False), ({"M": 64, "N": 51160, "K": 4317}, False),              # a B from HBM that no copy would touch, two rounds of workgroups
    ({"M": 40, "N": 30976, "K": 7889}, True), ({"M": 40, "N": 63977, "K": 1001, "tn": True}, True),                  # ... one round; a B that would be copied
    ({"M": 395, "N": 1831, "K": 3883}, False), ({"M": 2000, "N": 1901, "K": 2001}, False),   # long unsplit K from HBM
    ({"M": 395, "N": 1831, "K": 383}, True)])
def test_in_place_off_the_grid_only_where_it_is_not_slower_from_memory_either(q, in_place):
    """Problems that reading in place made up to 1.6 times slower once their operands are not in the cache keep their copies."""
    (r,) = ask([q])
    assert r["run"] == 0 and (",di=1" in r["describe"]) == in_place, r["describe"]


@pytest.mark.parametrize("m", [1, 4, 16, 32])
def test_few_rows_of_a_fit_the_static_scratch_and_keep_in_place_kernels_off_the_grid(m):
    """What the static entry point takes with few rows is the planned call; operands that would be copied are still read where they lie."""
    on = [{"M": m, "N": n, "K": k, "tn": tn} for n in (1000, 5480, 13736, 40008, 64000) for k in (512, 2360, 5152, 12912) for tn in (False, True)]
    for q, r in zip(on, ask(on)):
        assert r["plan"] == 0 and r["run"] == 0 and r["workspace"] <= hg.STATIC_SCRATCH_BYTES, (q, r["describe"], r["workspace"])
        assert r["static"] == 0 and r["static_log"] == r["run_log"], (q, r["describe"])
    off = [{"M": m, "N": n, "K": k, "tn": True} for n, k in [(1729, 1545), (6747, 2667), (3137, 957), (35783, 3107)]]
    for q, r in zip(off, ask(off)):
        assert ",di=1" in r["describe"], (q, r["describe"])


def test_streaming_rows_of_the_table_do_not_keep_a_b_off_the_grid_from_being_read_where_it_lies():
    """Next to a row of the column-major table that names the streaming family: no copy of B.  Where B can be read as it is (only A, or C, is off the
    grid), the row stands."""
    shapes = [s for s, spec in table_rows(True) if spec.startswith("skinny")]
    assert len(shapes) > 10
    off = [{"M": m, "N": n - dn, "K": k - dk, "tn": True, **({"ldb": k + db} if db else {})} for m, n, k in shapes for dn, dk, db in ((0, 1, 0), (0, 4, 0), (3, 5, 0), (0, 0, 1), (0, 0, 4))]
    for q, r in zip(off, ask(off)):
        assert ",di=1" in r["describe"] and "pad_copy" not in str(r["run_log"]), (q, r["describe"])
    read = [{"M": m, "N": n - dn, "K": k, "tn": True, **more} for m, n, k in shapes for dn, more in ((1, {}), (4, {}), (0, {"lda": k + 1}), (0, {"ldc": n + 1}))]
    for q, r in zip(read, ask(read)):
        assert r["describe"].startswith("skinny,") and len([k for k in kernels(r["run_log"]) if k[0] != "pad_copy_kernel"]) == 1, (q, r["describe"])


def test_the_reported_workgroups_are_those_of_the_launch():
    """Strips with several blocks of rows are launched in whole rounds of the XCDs."""
    qs = [{"M": m, "N": n, "K": 2048, "tn": tn} for m, n, tn in ((17, 2040, True), (96, 3000, True), (320, 640, True), (65, 2504, False), (17, 1000, False), (16, 4096, True), (8, 5000, True),
                                                                 (512, 512, False), (3, 30000, True))]
    for q, r in zip(qs, ask(qs)):
        name, x, y, *_ = kernels(r["run_log"])[0]
        assert r["workgroups"] == x * y, (q, r)


@pytest.mark.parametrize("m,n,k,tn", [(95, 3856, 2840, True), (218, 576, 3312, True), (282, 1288, 3568, True), (46, 1344, 6144, True), (97, 576, 6016, True), (128, 520, 2048, False),
                                      (64, 2040, 2048, True)], ids=str)
def test_blocks_of_rows_in_strips_are_one_workgroup_for_every_compute_unit(m, n, k, tn):
    """... of each XCD, which workgroups go round: as many are launched as there are tiles, so that none of 32 compute units holds two."""
    (r,) = ask([{"M": m, "N": n, "K": k, "tn": tn}])
    nr, mr = (int(re.search(rf"{key}=(\d+)", r["describe"])[1]) for key in ("nr", "mr"))
    ((_, x, y, *_),) = kernels(r["run_log"])
    assert x * y == -(-m // mr) * -(-n // nr) <= 256 and y == 1, (x, y, r["describe"])
