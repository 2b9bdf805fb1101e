"""The range in which the planner takes one strip of a column-major B for every compute unit (no GPU)."""
import pytest

import paper_2512_02551_amd as hg
from fake_hip import ask
from paper_2512_02551_amd import strips

MEASURED = strips.load([strips.CHECK])
ERR_INVALID_ARG, ERR_UNSUPPORTED = 1, 2


def picked(m, n, k, **layout):
    return hg.plan_choice(m, n, k, hg.Layouts.make(b_col_major=True, **layout)).split(": ", 1)[-1]


@pytest.mark.parametrize("m,n,k,spec", [
    (1, 4096, 4096, "skinny,sk=1"), (16, 4096, 16384, "skinny,sk=1"), (32, 4096, 4992, "skinny,sk=1"), (16, 11008, 4088, "skinny,sk=1,nr=48"),
    (16, 4112, 5200, "skinny,sk=1,nr=32"), (4, 8192, 28672, "skinny,sk=1,nr=32"), (2, 12288, 768, "skinny,sk=1,nr=48"), (8, 512, 6240, "skinny,sk=1")], ids=str)
def test_inside(m, n, k, spec):
    assert picked(m, n, k) == spec
    assert picked(m, n, k, lda=k + 64, ldb=k + 8, ldc=n + 8) == spec


@pytest.mark.parametrize("m,n,k", [
    (33, 4096, 4096), (16, 12304, 4096), (16, 4104, 4096), (16, 4095, 4096), (16, 4096, 4095), (32, 4096, 5008), (16, 4112, 5216), (8, 512, 6256), (4, 12288, 760),
    (16, 512, 512)], ids=str)
def test_outside(m, n, k):
    """More rows, more columns or columns off 16, a longer K, a shorter one, a pick whose calls share launches."""
    assert picked(m, n, k) != "skinny,sk=1" + {1: "", 2: ",nr=32", 3: ",nr=48", 4: ",nr=64"}[-(-n // 4096)]


def test_row_major_b_is_not_touched():
    assert "nr=" not in hg.plan_choice(16, 11008, 4096) and hg.plan_choice(16, 4096, 4096).startswith("table: mfma,")


@pytest.mark.parametrize("m,n,k,tile", [
    (17, 2048, 6144, (16, 16)), (32, 64, 4608, (16, 16)), (33, 4096, 4096, (32, 32)), (64, 2048, 4096, None), (40, 2048, 4096, (32, 16)), (48, 8192, 3584, (32, 48)),
    (64, 4000, 4096, (32, 32)), (96, 3072, 3584, (48, 32)), (320, 640, 3072, (32, 32)), (129, 1160, 2048, (32, 32))], ids=str)
def test_blocks_of_rows_inside(m, n, k, tile):
    """The fewest rows of A and B together that one workgroup for every compute unit covers; a table's row stays."""
    assert ("mr=" not in picked(m, n, k)) if tile is None else picked(m, n, k, lda=k + 64, ldb=k + 8, ldc=n + 8) == "skinny,sk=1,nr=%d,mr=%d" % tile


@pytest.mark.parametrize("m,n,k", [
    (16, 2048, 4096), (17, 2064, 4096), (17, 2056, 4096), (17, 2048, 6152), (32, 32, 4616), (33, 4096, 4104), (48, 8192, 3592), (64, 8192, 2048), (64, 4001, 4096),
    (64, 4000, 4095), (64, 4000, 1016), (72, 5000, 1272), (321, 640, 3072), (320, 632, 3080)], ids=str)
def test_blocks_of_rows_outside(m, n, k):
    """Fewer rows, more tiles than compute units, a longer K, a shorter one, sizes off 8, more rows than twice the columns."""
    assert "mr=" not in picked(m, n, k)


def statuses(specs, **q):
    return [r["plan"] for r in ask([{**q, "spec": s} for s in specs])]


def test_which_blocks_of_rows_there_are():
    """Of a column-major B 16 to 64 rows in steps of 16, without a split; other values are no specs, and some waves have no kernel."""
    taken = ["skinny,sk=1,mr=16", "skinny,sk=1,mr=64", "skinny,sk=1,nr=16,mr=48", "skinny,sk=1,nr=64,mr=64", "skinny,sk=1,wv=16,nr=32,mr=32", "skinny,sk=1,fr=1,mr=16"]
    assert statuses(taken, M=64, N=4096, K=4096, tn=True) == [0] * len(taken)
    invalid = ["skinny,sk=2,mr=16", "skinny,sk=1,mr=8", "skinny,sk=1,mr=24", "skinny,sk=1,mr=80", "skinny,sk=1,wv=8,ra=1,mr=16", "mfma,bm=32,bn=64,bk=64,wm=1,wn=2,st=4,pf=3,sk=1,gm=8,mr=16"]
    assert statuses(invalid, M=64, N=4096, K=4096, tn=True) == [ERR_INVALID_ARG] * len(invalid)
    assert statuses([invalid[-1][:-6]], M=64, N=4096, K=4096, tn=True) == statuses(["skinny,sk=1,wv=8,ra=1"], M=32, N=4096, K=4096, tn=True) == [0]
    missing = ["skinny,sk=1,wv=16,nr=16,mr=48", "skinny,sk=1,wv=16,nr=64,mr=32", "skinny,sk=1,wv=8,nr=48,mr=64"]
    assert statuses(missing, M=64, N=4096, K=4096, tn=True) == [ERR_UNSUPPORTED] * len(missing)


def test_which_blocks_of_rows_there_are_for_a_row_major_b():
    taken = ["skinny,sk=1,nr=32,mr=16", "skinny,sk=1,nr=32,mr=32"]
    assert statuses(taken, M=17, N=4096, K=2048) == [0, 0]
    missing = ["skinny,sk=1,mr=16", "skinny,sk=1,nr=16,mr=16", "skinny,sk=1,nr=64,mr=16", "skinny,sk=1,nr=32,mr=48", "skinny,sk=1,nr=32,mr=64", "skinny,sk=1,wv=8,nr=32,mr=16"]
    assert statuses(missing, M=17, N=4096, K=2048) == [ERR_UNSUPPORTED] * len(missing)


def test_row_major_strips_up_to_31_bits_of_offset():
    """Copies of the last chunk reach up to 256 rows past K; problems that come with such a pitch have 512 rows past it below 2 GiB."""
    for k in (2048, 1536):
        ldb = ((1 << 30) // (k + 512) - 1) // 8 * 8
        assert (k + 512) * ldb * 2 < 1 << 31 <= (k + 512) * (ldb + 8) * 2
        inside, outside = ask([{"M": 17, "N": 1024, "K": k, "ldb": x, "spec": "skinny,sk=1,nr=32,mr=16"} for x in (ldb, ldb + 8)])
        assert (inside["plan"], outside["plan"]) == (0, ERR_UNSUPPORTED)
        inside, outside = ask([{"M": 17, "N": 1024, "K": k, "ldb": x} for x in (ldb, ldb + 8)])
        assert "mr=16" in inside["describe"] and "mr=" not in outside["describe"] and outside["plan"] == 0


@pytest.mark.parametrize("m,n,k,mr", [(17, 4096, 2048, 16), (32, 4032, 1536, 16), (64, 1920, 2048, 16), (65, 2504, 1776, 32), (96, 2560, 2048, 32)], ids=str)
def test_row_major_b_inside(m, n, k, mr):
    got = hg.plan_choice(m, n, k, hg.Layouts.make(lda=k + 64, ldb=n + 8, ldc=n + 8))
    assert got.split(": ", 1)[1] == f"skinny,sk=1,nr=32,mr={mr}"


@pytest.mark.parametrize("m,n,k,pad", [(16, 4096, 2048, 8), (17, 4104, 2048, 8), (17, 4096, 2056, 8), (17, 4096, 760, 8), (97, 2560, 2048, 8), (321, 256, 1024, 8), (320, 632, 1536, 8),
                                       (17, 4095, 2048, 8), (17, 4096, 2048, 1), (17, 4096, 2048, 1 << 20)], ids=str)
def test_row_major_b_outside(m, n, k, pad):
    """Fewer rows, more tiles than compute units, a longer K, a shorter one, more rows, sizes off 8, a B whose offsets leave 31 bits."""
    assert "mr=" not in hg.plan_choice(m, n, k, hg.Layouts.make(lda=k + 64, ldb=n + pad, ldc=n + 8))


def test_a_default_width_never_refuses_what_strips_of_16_rows_take():
    """A spec without nr: the strips that fill the compute units as far as waves and blocks of A have such a kernel, narrower ones where not."""
    qs = [{"M": m, "N": n, "K": k, "tn": True, "spec": f"skinny,sk={sk}" + (",fr=1" if fr else "") + (f",wv={wv}" if wv != 4 else "")}
          for m in (1, 16, 17, 32, 33, 64) for n in (4096, 4104, 8192, 8200, 12288, 12296, 16384, 16392) for wv in (4, 8, 16)
          for k, sk, fr in ((1024, 1, 0), (2048, 2, 0), (2048, 2, 1), (64, 2, 0), (64, 3, 1))]
    wide = 0
    for q, r, sixteen in zip(qs, ask(qs), ask([{**q, "spec": q["spec"] + ",nr=16"} for q in qs])):
        assert sixteen["plan"] == 0 and r["plan"] == 0 and r["run"] == 0, (q, r)
        wide += r["run_log"] != sixteen["run_log"]
    assert wide > 100
    # the widest strips that 8 waves times four blocks of A, and 16 waves times two, have kernels for
    for m, wv, width in ((64, 8, 32), (32, 16, 32), (64, 16, 16), (64, 4, 48), (32, 8, 48)):
        spec = f"skinny,sk=1,wv={wv}" if wv != 4 else "skinny,sk=1"
        plain, wide = ask([{"M": m, "N": 12288, "K": 1024, "tn": True, "spec": spec + x} for x in ("", f",nr={width}")])
        assert plain["plan"] == 0 and plain["run_log"] == wide["run_log"], (m, wv, plain)


@pytest.mark.parametrize("m,n,k,ldb,mr", [
    (17, 2048, 1416, 2048, 0), (17, 2048, 1408, 2048, 16), (17, 2048, 2048, 2056, 16), (20, 2048, 2048, 2048, 0), (64, 1792, 2048, 2560, 0), (64, 1792, 2048, 1792, 16),
    (24, 1528, 1536, 2560, 16), (24, 1536, 1536, 1536, 0), (65, 1536, 2048, 1536, 16), (64, 1024, 2048, 1024, 16), (65, 2560, 2048, 2560, 32)], ids=str)
def test_row_major_b_whose_half_lines_come_slowly(m, n, k, ldb, mr):
    """Few blocks of rows on a wide B whose rows are a multiple of 1 KiB apart: what was up to 1.2 times slower from HBM."""
    got = hg.plan_choice(m, n, k, hg.Layouts.make(ldb=ldb, ldc=n + 8))
    assert got.split(": ", 1)[1] == f"skinny,sk=1,nr=32,mr={mr}" if mr else "mr=" not in got, got


@pytest.mark.parametrize("spec", ["skinny,sk=1,nr=32,mr=16", "skinny,sk=1,mr=64", "skinny,sk=1,wv=8,nr=16,mr=32", "skinny,sk=1,wv=8,ra=1"])
def test_no_model_describes_blocks_of_rows_or_resident_a(spec):
    with pytest.raises(hg.HgemmError) as e:
        hg.predict_us(64, 2048, 2048, spec)
    assert e.value.status == ERR_UNSUPPORTED
    assert hg.predict_us(64, 2048, 2048, "skinny,sk=1") > 1.0


@pytest.mark.parametrize("kind,count,most_slower", [("row-major B", 1000, 0.05), ("blocks of rows", 2700, 0.03), ("all rows", 3700, 0.04)])
def test_limits_on_measured_problems(kind, count, most_slower):
    """Strips where they are faster than the kernels chosen without them, from HBM and from the cache; what they are not taken for is level or slower from HBM, on average."""
    rows = [r for r in MEASURED if kind == ("row-major B" if not r["tn"] else "blocks of rows" if "mr=" in r["strips"] else "all rows")]
    taken = [r for r in rows if strips.takes(r)]
    left = [r for r in rows if not strips.takes(r)]
    n, hbm, cache, slower, slower_cache, *_ = strips.figures(taken)
    assert n >= count and hbm < 0.83 and cache < 0.75 and slower < most_slower * n and slower_cache < 0.015 * n, strips.figures(taken)
    assert strips.figures(left)[1] > 0.95, strips.figures(left)
