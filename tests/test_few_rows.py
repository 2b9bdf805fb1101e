"""Measured problems behind the choice for few rows of A (no GPU): the committed rows are what the committed timings give, every row can be
looked up, and the built library's choices on those timings are close to the fastest kernel from HBM and from the cache."""
import re

import numpy as np
import pytest

import paper_2512_02551_amd as hg
from paper_2512_02551_amd import few_rows as fr


@pytest.fixture(scope="module")
def timings():
    return fr.load([fr.DATA])


@pytest.fixture(scope="module")
def check():
    return fr.load([fr.CHECK])


@pytest.fixture(scope="module")
def committed():
    text = open(fr.INC).read()
    specs = re.findall(r'^    "([^"]+)",$', text, re.M)
    rows = {}
    for tn, name in ((False, "kFewRowsNN"), (True, "kFewRowsTN")):
        part = text[text.index(name):].split("};", 1)[0]
        rows[tn] = [(tuple(map(int, m[:3])), [specs[int(i)] for i in m[3].split(",") if int(i) >= 0]) for m in re.findall(r"\{(\d+), (\d+), (\d+), \{([^}]*)\}\}", part)]
    return specs, rows


def test_rows_are_of_few_rows_in_search_order_and_within_reach(committed):
    specs, rows = committed
    assert len(specs) <= 127 and len(set(specs)) == len(specs)
    for tn, r in rows.items():
        assert len(r) > 1500
        assert [fr.columns_quarter(s[1]) for s, _ in r] == sorted(fr.columns_quarter(s[1]) for s, _ in r)
        assert all(a[0][2] <= b[0][2] for a, b in zip(r, r[1:]) if fr.columns_quarter(a[0][1]) == fr.columns_quarter(b[0][1]))
        for (m, n, k), listed in r:
            assert 1 <= m <= 32 and n % 8 == 0 and k % 8 == 0 and 1 <= len(listed) <= fr.LISTED == len(set(listed)) + fr.LISTED - len(listed)
            assert tn or 2.0 * n * k < 2 ** (28 + fr.REACH)              # a longer row-major B is streamed


def test_committed_rows_are_built_from_the_committed_timings(timings, committed, tmp_path):
    fr.write(fr.build(timings), "", str(tmp_path / "rows.inc"))
    a, b = open(fr.INC).read().split("\n", 3), open(tmp_path / "rows.inc").read().split("\n", 3)
    assert a[3] == b[3]                                                 # the third line says what they were built from


def test_choices_on_other_problems_are_close_to_the_fastest_kernel(check):
    ratios = []
    for r in check:
        t = {c[0]: c[1:] for c in r["cands"]}
        s = fr.choice(None, *r["shape"], r["tn"])
        if s in t:
            ratios.append([t[s][w] / min(v[w] for v in t.values()) for w in (0, 1)])
    ratios = np.array(ratios)
    assert len(ratios) > 0.99 * len(check)
    hbm, cache = np.exp(np.log(ratios).mean(axis=0))
    assert hbm < 1.06 and cache < 1.08, (hbm, cache)


@pytest.mark.parametrize("m,n,k,tn,not_taken", [
    (24, 18368, 1088, False, "bn=192"), (31, 12496, 2336, False, "bn=128"), (28, 20296, 1928, False, "bn=192"), (31, 10424, 1488, False, "bn=128"),    # what 33 rows and more take
    (1, 30144, 2112, True, "ra=1"), (15, 31736, 2528, True, "ra=1"), (9, 26504, 2504, True, "ra=1"),
    (21, 6272, 1408, True, "ra=1"), (21, 5760, 1664, True, "ra=1"), (21, 7168, 1792, True, "ra=1")])               # level from HBM, slower from the cache
def test_few_rows_do_not_take(m, n, k, tn, not_taken):
    """Kernels that were up to 1.35 times slower than the models' picks."""
    choice = hg.plan_choice(m, n, k, hg.Layouts.make(b_col_major=tn))
    assert not re.search(not_taken, choice), choice
