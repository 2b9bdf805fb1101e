"""Up to 32 rows of A off the dispatch table: the kernels of the nearest measured problem (few_rows.inc)."""
import pytest

import paper_2512_02551_amd as hg
from test_gpu_direct import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,tn,kernel", [
    (1, 1008, 848, False, "mfma,bm=32,bn=64,bk=64"), (3, 912, 2928, False, "mfma,bm=32,bn=64,bk=64"), (31, 10424, 1488, False, "mfma,bm=32,bn=64,bk=64"), (31, 20480, 4992, False, "mfma,bm=32,bn=128,bk=128"),
    (10, 7944, 2248, False, "mfma,bm=32,bn=128,bk=64"), (7, 10592, 5880, False, "mfma,bm=32,bn=192,bk=64"), (23, 11960, 6120, False, "mfma,bm=32,bn=256,bk=64"),
    (1, 1072, 936, True, "skinny"), (15, 1035, 928, True, "mfma,bm=32,bn=64,bk=64"), (12, 4088, 952, True, "skinny,sk=1,wv=8,nr=32"), (4, 4720, 1200, True, "skinny,sk=1,nr=32"),
    (2, 845, 3768, True, "mfma,bm=32,bn=64,bk=64"), (14, 6029, 1552, True, "skinny,sk=1,wv=8,ra=1"), (16, 50257, 4096, True, "skinny,sk=1,wv=8,ra=1"), (8, 16761, 1032, True, "mfma,bm=32,bn=128,bk=128"),
    (3, 2837, 8344, True, "mfma,bm=32,bn=128,bk=64"), (3, 6776, 6384, True, "mfma,bm=32,bn=192,bk=64"), (32, 40005, 1304, True, "skinny,sk=1,wv=8,ra=1"),
    (16, 16384, 1200, True, "skinny,sk=1,wv=8,ra=1"), (1, 20001, 4096, True, "skinny,sk=1,wv=8,ra=1"), (16, 16392, 4104, True, "mfma")], ids=str)
def test_the_measured_pick_is_exact_on_small_integers_and_stays_inside_c(m, n, k, tn, kernel):
    assert check(None, m, n, k, tn).startswith(kernel)


RESIDENT = "skinny,sk=1,wv=8,ra=1"


@pytest.mark.parametrize("m,n,k", [
    (1, 8, 8), (16, 16, 256), (3, 24, 264), (15, 4096, 1536), (16, 4112, 1544), (9, 8200, 2048), (1, 4104, 2056), (16, 4360, 3072), (7, 12296, 3080), (16, 4096, 4096),
    (2, 4120, 4104), (16, 4136, 5120), (5, 4128, 5128), (16, 8192, 8192), (17, 8, 264), (32, 4104, 1536), (31, 8208, 1800), (17, 4112, 2048), (20, 4200, 2568), (32, 12304, 3080), (32, 4096, 4096)],
    ids=str)
def test_a_resident_in_registers(m, n, k):
    """Fewer strips than workgroups, whole and ragged rounds of them, half a strip, every instance at the largest K it takes and 8 more
    than the one before takes; NaN between the rows of A, B and C and behind them; infinities and NaN in A and B."""
    assert check(RESIDENT, m, n, k, True) == RESIDENT
    check(RESIDENT, m, n, k, True, (8, 16, 8), (8, 8, 8), special=True)


def test_a_resident_in_registers_is_refused_where_no_instance_holds_it():
    for m, n, k, tn in [(33, 4096, 1024, True), (16, 4096, 8200, True), (17, 4096, 4104, True), (16, 4096, 1024, False)]:
        with pytest.raises(hg.HgemmError):
            hg.Plan(m, n, k, hg.Layouts.make(b_col_major=tn), RESIDENT)
    for spec in ("skinny,sk=2,wv=8,ra=1", "skinny,sk=1,ra=1", "skinny,sk=1,wv=8,nr=32,ra=1", "skinny,sk=1,wv=8,ra=2", "mfma,bm=32,bn=64,bk=64,wm=1,wn=2,st=4,pf=3,ra=1"):
        with pytest.raises(hg.HgemmError):
            hg.Plan(16, 4096, 1024, hg.Layouts.make(b_col_major=True), spec)
