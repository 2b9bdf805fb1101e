"""Up to 32 rows of A off the dispatch table: the kernels of the nearest measured problem (few_rows.inc)."""
import pytest

from test_gpu_direct import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,tn,kernel", [
    (1, 1008, 848, False, "mfma,bm=32,bn=64,bk=64"), (3, 912, 2928, False, "mfma,bm=32,bn=64,bk=64"), (31, 10424, 1488, False, "mfma,bm=32,bn=128,bk=128"),
    (10, 7944, 2248, False, "mfma,bm=32,bn=128,bk=64"), (7, 10592, 5880, False, "mfma,bm=32,bn=192,bk=64"), (23, 11960, 6120, False, "mfma,bm=32,bn=256,bk=64"),
    (1, 1072, 936, True, "skinny"), (15, 1035, 928, True, "skinny"), (12, 4088, 952, True, "skinny,sk=1,wv=8,nr=32"), (4, 4720, 1200, True, "skinny,sk=1,nr=32"),
    (2, 845, 3768, True, "mfma,bm=32,bn=64,bk=64"), (14, 6029, 1552, True, "mfma,bm=32,bn=64,bk=64"), (8, 16761, 1032, True, "mfma,bm=32,bn=128,bk=128"),
    (3, 2837, 8344, True, "mfma,bm=32,bn=128,bk=64"), (3, 6776, 6384, True, "mfma,bm=32,bn=192,bk=64"), (32, 40005, 1304, True, "")], ids=str)
def test_the_measured_pick_is_exact_on_small_integers_and_stays_inside_c(m, n, k, tn, kernel):
    assert check(None, m, n, k, tn).startswith(kernel)
