"""When the cost model picks the fused split-K reduction (no GPU)."""
import pytest

import paper_2512_02551_amd as hg


@pytest.mark.parametrize("m,n,k,tn", [(33, 64, 8192, False), (69, 64, 10272, False), (101, 72, 2184, True), (68, 200, 920, True), (119, 120, 1456, True)], ids=str)
def test_never_beyond_32_rows(m, n, k, tn):
    assert "fr=1" not in hg.plan_choice(m, n, k, hg.Layouts.make(b_col_major=tn))


def test_up_to_32_rows_it_stays():
    assert "fr=1" in hg.plan_choice(32, 64, 8192) and "fr=1" in hg.plan_choice(8, 520, 3104)
