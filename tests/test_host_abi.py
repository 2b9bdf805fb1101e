"""CPU-only checks: the library loads, exports every declared symbol, and its host-side logic
(tile arithmetic, tile order) is right.  No kernel is launched here."""
import os
import re

import pytest

import paper_2512_02551_amd as hg

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(hg.lib_path()):
        from paper_2512_02551_amd import build
        build.build(force=True)
    return hg.load()


def test_every_declared_symbol_is_exported(lib):
    header = open(os.path.join(ROOT, "include", "hgemm.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(hgemm_[a-z_]+)\s*\(", header))
    assert declared == set(hg.EXPORTS)
    for name in declared:
        assert hasattr(lib, name), name


def test_status_strings(lib):
    for s in range(6):
        assert hg.status_string(s)
    assert "gfx950" in hg.status_string(5)


def test_run_entry_points_refuse_a_null_plan_before_touching_the_gpu(lib):
    import ctypes
    one = (ctypes.c_void_p * 1)(0)
    assert lib.hgemm_run(None, None, None, None, None) == 1
    assert lib.hgemm_run_many(None, 1, 1, 0, one, one, one, None) == 1


def test_padding_arithmetic_matches_the_papers_example(lib):
    # Section 5.2: M = 8192, BM = 160 -> 52 tiles, 8320 rows
    assert hg.tiles(8192, 160) == 52
    assert hg.padded(8192, 160) == 8320
    assert hg.tiles(0, 64) == 0 and hg.tiles(1, 64) == 1 and hg.tiles(64, 64) == 1 and hg.tiles(65, 64) == 2
    assert hg.tiles(5, 0) == -1


@pytest.mark.parametrize("tm,tn", [(1, 1), (3, 5), (32, 32), (16, 16), (40, 35), (7, 300), (300, 7), (64, 43), (1, 1000)])
@pytest.mark.parametrize("group", [0, 1, 3, 8, 16])
def test_tile_order_is_a_bijection(lib, tm, tn, group):
    total = tm * tn
    seen = [hg.tile_of_workgroup(w, tm, tn, group) for w in range(total)]
    assert sorted(seen) == list(range(total))
    assert hg.tile_of_workgroup(total, tm, tn, group) == -1


def test_tile_order_keeps_an_xcd_on_a_compact_block(lib):
    # 32 x 32 tiles, group 8: the 32 workgroups one XCD gets from a run of 256 ids
    # (ids congruent mod 8) must cover 8 tile-rows x 4 tile-columns.
    tm = tn = 32
    for xcd in range(8):
        tiles = [hg.tile_of_workgroup(w, tm, tn, 8) for w in range(xcd, 256, 8)]
        rows = {t // tn for t in tiles}
        cols = {t % tn for t in tiles}
        assert len(rows) == 8 and len(cols) == 4
    # and a whole run of 256 ids covers 8 rows x 32 columns
    tiles = [hg.tile_of_workgroup(w, tm, tn, 8) for w in range(256)]
    assert {t // tn for t in tiles} == set(range(8)) and {t % tn for t in tiles} == set(range(32))


def test_candidates_and_help_are_consistent(lib):
    specs = hg.candidates(4096, 4096, 4096)
    assert specs and all(s.startswith("mfma,") for s in specs)
    assert hg.candidates(3, 5, 7) == ["generic"]
    text = hg.spec_help()
    assert "generic" in text and "mfma" in text
    skinny = hg.candidates(16, 4096, 4096)
    assert any("sk=8" in s or "sk=16" in s for s in skinny)


# ---- randomised host-side properties ----------------------------------------------------------------

from hypothesis import given, settings, strategies as hst  # noqa: E402


@settings(max_examples=60, deadline=None)
@given(tm=hst.integers(1, 70), tn=hst.integers(1, 70), group=hst.sampled_from([0, 1, 2, 3, 4, 8, 16, 64]))
def test_tile_order_is_a_permutation_for_random_grids(tm, tn, group):
    import paper_2512_02551_amd as hg
    seen = sorted(hg.tile_of_workgroup(w, tm, tn, group) for w in range(tm * tn))
    assert seen == list(range(tm * tn))
    assert hg.tile_of_workgroup(tm * tn, tm, tn, group) == -1            # one past the end is refused


@settings(max_examples=200, deadline=None)
@given(dim=hst.integers(0, 1 << 24), tile=hst.sampled_from([8, 32, 64, 128, 160, 256]))
def test_padding_arithmetic_properties(dim, tile):
    import paper_2512_02551_amd as hg
    t, p = hg.tiles(dim, tile), hg.padded(dim, tile)
    assert p == t * tile and p >= dim and p - dim < tile


@settings(max_examples=40, deadline=None)
@given(M=hst.integers(1, 20000), N8=hst.integers(1, 2500), K8=hst.integers(1, 2500))
def test_every_candidate_has_a_finite_positive_prediction(M, N8, K8):
    """The planner takes the minimum of the cost model over these candidates, so the model has to be
    defined (finite, positive) on every one of them, for any aligned shape."""
    import math

    import paper_2512_02551_amd as hg
    N, K = 8 * N8, 8 * K8
    cands = [s for s in hg.candidates(M, N, K) if "sm=1" not in s and "tb=1" not in s and "ps=1" not in s]
    assert cands and all(s.startswith(("mfma,", "skinny,")) for s in cands)
    for s in cands[::3]:
        us = hg.predict_us(M, N, K, s)
        assert math.isfinite(us) and us > 1.0, (M, N, K, s, us)


def test_plan_choice_names_the_source_of_every_kind_of_plan():
    """hgemm_plan_choice is the planner's decision without a device: dispatch table, nearest tuned shape for large
    problems off the table (unless its tiles fill the last round of workgroups worse than the model's pick),
    cost model, streaming family for a few rows against weights no cache holds, padded copies, blocks for
    operands of 2 GiB and more, generic kernel."""
    import workloads as wl
    tn = hg.Layouts.make(b_col_major=True)
    for s in [wl.C1_SHAPE, *wl.C2_SHAPES, *wl.C3_SHAPES, *wl.C5_SHAPES, *wl.c4_shapes()[::7]]:
        assert hg.plan_choice(*s).startswith("table: "), s
        assert hg.plan_choice(*s, tn).startswith("table: "), s
    assert hg.plan_choice(16, 28672, 8192) == "table: skinny,sk=1"
    assert hg.plan_choice(1, 4096, 4096, tn).startswith("table: skinny,")        # column-major B has streaming rows of its own
    assert hg.plan_choice(1, 15360, 5120).startswith("table: skinny,") and hg.plan_choice(1, 15360, 5120, tn).startswith("table: mfma,")
    near = hg.plan_choice(3000, 5120, 5120)
    assert near.startswith("neighbour: mfma,bm=256,bn=256,") and "mi=16" in near
    assert hg.plan_choice(3000, 6144, 4096).startswith("model: mfma,bm=192,bn=192,")      # 512 tiles against the neighbour's 288
    assert hg.plan_choice(4096, 4096, 4096, hg.Layouts.make(lda=4104)).startswith(("neighbour: ", "model: "))   # not packed: no table row
    assert hg.plan_choice(8, 16384, 8192).startswith("model: skinny,")
    assert hg.plan_choice(8, 4096, 4096).startswith("model: mfma,")
    assert hg.plan_choice(300, 264, 128).startswith("model: mfma,")
    assert hg.plan_choice(1000, 1001, 1003).endswith(",pad=1")
    assert hg.plan_choice(100, 100, 100) == "generic" and hg.plan_choice(0, 5, 5) == "empty"
    assert hg.plan_choice(32768, 32768, 32768) == "blocks,rows=16384,cols=16384,bt=1"
    assert hg.plan_choice(32768, 32768, 32768, tn) == "blocks,rows=16384,cols=16384"
    assert hg.plan_choice((1 << 21), 64, 1024) == "blocks,rows=699136,cols=64"
    with pytest.raises(hg.HgemmError):
        hg.plan_choice(-1, 8, 8)
    with pytest.raises(hg.HgemmError):
        hg.plan_choice(64, 64, 64, hg.Layouts.make(lda=8))


def test_plan_choice_is_the_same_from_every_thread_and_after_many_other_shapes():
    """The cost model's picks are kept per thread in a table of 64: a shape asked again, asked after many others took its
    place, and asked from a thread that has never planned gets one answer, in both layouts."""
    import random
    import threading

    rnd = random.Random(17)
    shapes = [(rnd.randint(1, 3000), 8 * rnd.randint(1, 400), 8 * rnd.randint(1, 400), rnd.random() < 0.5) for _ in range(300)]

    def ask(out):
        for m, n, k, tn in shapes:
            out.append(hg.plan_choice(m, n, k, hg.Layouts.make(b_col_major=tn)))

    first, again, other = [], [], [[] for _ in range(4)]
    ask(first)
    ask(again)
    threads = [threading.Thread(target=ask, args=(o,)) for o in other]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert first == again and all(o == first for o in other)
    for i in (0, 150, 299):                                    # asked twice in a row: the second answer comes from the table
        m, n, k, tn = shapes[i]
        lay = hg.Layouts.make(b_col_major=tn)
        assert hg.plan_choice(m, n, k, lay) == hg.plan_choice(m, n, k, lay) == first[i]


@pytest.mark.parametrize("spec", ["", "mfma,", "mfma,bm", "mfma,bm=", "mfma,bm=64x", "mfma,=3", "mfma,bm=64,,bn=64", "mfmax", "mfma;bm=64", "skinny,sk=0",
                                  "mfma,bm=-1", "mfma,zz=1", "mfma,bm=99999999", "skinny,wv=5", "mfma,ph=2", "skinny,ph=1", "mfma,bm=64,"])
def test_malformed_specs_are_invalid_arguments(spec):
    with pytest.raises(hg.HgemmError) as e:
        hg.predict_us(64, 64, 64, spec)
    assert e.value.status == 1, spec


def test_phased_kernels_take_over_large_problems_off_the_table():
    """A pick of the cost model or of the nearest tuned shape gives way to a phased kernel where one is predicted clearly
    faster, or keeps its tile and takes the phased schedule; short K and cache-line straddling rows of B keep the pick."""
    import random
    import re

    tn = hg.Layouts.make(b_col_major=True)
    assert "ph=1" in hg.plan_choice(9306, 2632, 10032, tn) and "ph=1" in hg.plan_choice(2746, 10800, 7456, tn)
    assert "ph=1" not in hg.plan_choice(1595, 8232, 104) and "ph=1" not in hg.plan_choice(776, 4056, 2656)
    rnd = random.Random(23)
    phased = 0
    for _ in range(1500):
        m, n, k = rnd.randint(96, 9000), 8 * rnd.randint(12, 1200), 8 * rnd.randint(8, 1200)
        lay = hg.Layouts.make(b_col_major=rnd.random() < 0.5)
        spec = hg.plan_choice(m, n, k, lay).split(": ")[1]
        if "ph=1" not in spec:
            continue
        phased += 1
        kv = {a: int(b) for a, b in re.findall(r"(\w+)=(\d+)", spec)}
        assert kv["bm"] < 2 * m and kv["bn"] < 2 * n and k // kv["sk"] >= 128, (m, n, k, spec)
        assert "sm=1" not in spec and "ps=1" not in spec and "fr=1" not in spec and hg.predict_us(m, n, k, spec) > 1.0
    assert phased > 200


@pytest.mark.parametrize("m,n,k,ldb,phased", [(2048, 2048, 1008, 2056, False), (2048, 2048, 1003, 2056, False), (2048, 2048, 1003, 2048, True),
                                              (2048, 2040, 1003, 2048, True), (2048, 2040, 1008, 2048, True), (2048, 2041, 1003, 2056, True),
                                              (2048, 2033, 1003, 2048, False)])
def test_phased_choice_looks_at_the_pitch_the_kernel_reads_b_with(m, n, k, ldb, phased):
    """128 columns of a row-major B are phased where its rows start on cache lines: the caller's pitch where B is read in
    place, also beside a copied A, else that of its packed copy (2048 for 2041 columns, 2040 for 2033)."""
    choice = hg.plan_choice(m, n, k, hg.Layouts.make(ldb=ldb))
    assert "bm=128,bn=128" in choice and ("ph=1" in choice) == phased, choice


def test_a_phased_neighbour_keeps_the_row_by_row_order_on_whole_rounds_of_xcds_only():
    """gm = 0 is taken over from the nearest tuned shape where the columns of tiles are a multiple of eight."""
    import random
    import re

    rnd = random.Random(29)
    kept = dropped = 0
    for _ in range(3000):
        m, n, k = rnd.randint(512, 4000), 8 * rnd.randint(500, 2000), 8 * rnd.randint(40, 700)
        choice = hg.plan_choice(m, n, k)
        if not choice.startswith("neighbour") or "ph=1" not in choice:
            continue
        kv = {a: int(b) for a, b in re.findall(r"(\w+)=(\d+)", choice)}
        whole = -(-n // kv["bn"]) % 8 == 0
        assert kv["gm"] != 0 or whole, (m, n, k, choice)
        kept += kv["gm"] == 0
        dropped += not whole
    assert kept > 10 and dropped > 100
    assert "gm=8" in hg.plan_choice(1297, 5392, 12336)


def test_kept_picks_are_told_apart_by_every_part_of_their_key():
    """The table of kept picks has 64 places: of 1500 pairs of problems that differ in one of M, N and K, some twenty share a
    place (the two layouts of one problem lie side by side).  Asked right after its pair, a problem gets the answer that a
    thread asked nothing else gives."""
    import random
    import threading

    def in_a_thread_of_its_own(*problems):
        out = []
        t = threading.Thread(target=lambda: out.extend(hg.plan_choice(m, n, k, hg.Layouts.make(b_col_major=tn)) for m, n, k, tn in problems))
        t.start()
        t.join()
        return out

    rnd = random.Random(41)
    for part in range(4):
        differ = 0
        for _ in range(1500):
            one = [rnd.randint(1, 400), 8 * rnd.randint(1, 200), 8 * rnd.randint(1, 200), rnd.random() < 0.5]
            if part == 3:              # few rows: the streaming family is the model's for a row-major B only
                one[:3] = rnd.randint(1, 32), 8 * rnd.randint(200, 2500), 8 * rnd.randint(100, 1000)
            two = list(one)
            two[part] = not one[3] if part == 3 else one[part] + 8 * rnd.randint(1, 150)
            alone = in_a_thread_of_its_own(two)
            first, after = in_a_thread_of_its_own(one, two)
            assert after == alone[0], (one, two)
            differ += first != after
        assert differ > (40 if part == 3 else 300), (part, differ)


def test_no_pick_without_a_workspace_becomes_a_phased_split():
    """Below 512 rows or columns no tuned neighbour steps in, so the pick that a phased kernel replaces is the cost model's
    best: a split may come of it only if that is one."""
    import random
    import re

    rnd = random.Random(43)
    splits = plain = 0
    while splits < 25 or plain < 25:
        m, n, k = rnd.randint(96, 511), 8 * rnd.randint(12, 2000), 8 * rnd.randint(100, 2000)
        if rnd.random() < 0.5:
            m, n = n, 8 * (m // 8)
        tn = rnd.random() < 0.5
        lay = hg.Layouts.make(b_col_major=tn)
        choice = hg.plan_choice(m, n, k, lay)
        if 2 * m * n * k < 3e10 or not choice.startswith("model") or "ph=1" not in choice:
            continue
        def modelled(s):                        # what the cost model chooses among: not the schedules it does not know
            kv = {a: int(b) for a, b in re.findall(r"(\w+)=(\d+)", s)}
            return s.startswith("mfma") and kv["gm"] == 8 and kv["pf"] <= kv["bk"] // 16 and not kv.keys() & {"sm", "tb", "ps", "fr", "ph", "mi"}

        best = min((hg.predict_us(m, n, k, s), s) for s in hg.candidates(m, n, k, lay) if modelled(s))[1]
        if "sk=1," in choice:
            plain += 1
        else:
            splits += 1
            assert "sk=1," not in best, (m, n, k, tn, choice, best)
