"""The range in which the planner takes one strip of a column-major B for every compute unit (no GPU)."""
import pytest

import paper_2512_02551_amd as hg


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
