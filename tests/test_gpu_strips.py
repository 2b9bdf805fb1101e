"""Column-major B and few rows of A: strips of B through LDS of each wave's own (skinny_tn_gemm_kernel)."""
import pytest

import paper_2512_02551_amd as hg
from test_gpu_direct import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr", [16, 32, 48, 64])
@pytest.mark.parametrize("wv", [4, 8, 16])
@pytest.mark.parametrize("m,n,k", [
    (1, 8, 8), (16, 16, 64), (7, 24, 72), (16, 200, 1000), (9, 4112, 264),         # one block of A: less than a chunk, a part of one, rows past the end
    (17, 40, 256), (32, 136, 520), (24, 2056, 1032),                                 # two
    (33, 72, 512), (64, 264, 776),                                                   # four
    (5, 40, 4104), (20, 24, 3080), (50, 40, 3144)], ids=str)                         # chunks that come round in the ring, of sixteen waves too
def test_every_instance(m, n, k, wv, nr):
    """K off the 64 of a chunk and off the chunks of all waves, columns off the strips and off 16, padded leading dimensions, and
    infinities and NaN in A and B; splits in two launches and fused."""
    blocks = (1 if m <= 16 else 2 if m <= 32 else 4) * (nr // 16)
    spec = "skinny,sk=%d%s" + (f",wv={wv}" if wv != 4 else "") + f",nr={nr}"
    if wv * blocks > 64 or (wv == 16 and blocks > 4):
        with pytest.raises(hg.HgemmError):
            hg.Plan(m, n, k, hg.Layouts.make(b_col_major=True), spec % (1, ""))
        return
    assert check(spec % (1, ""), m, n, k, True) == spec % (1, "")
    check(spec % (1, ""), m, n, k, True, (8, 16, 8), (8, 8, 8), special=True)
    check(spec % (2, ""), m, n, k, True, (8, 16, 8), (8, 8, 8))
    check(spec % (3, ",fr=1"), m, n, k, True)


@pytest.mark.parametrize("m,n,wv", [(9, 4096, 4), (9, 4112, 4), (64, 8200, 8), (32, 8200, 16), (64, 4104, 16), (40, 12288, 4), (20, 12296, 8)], ids=str)
def test_default_widths(m, n, wv):
    """Strips whose width follows from the columns, waves and rows of A."""
    spec = "skinny,sk=1" + (f",wv={wv}" if wv != 4 else "")
    assert check(spec, m, n, 264, True, (8, 8, 8), (0, 8, 8)) == spec


@pytest.mark.parametrize("m,n,k,nr", [(1, 4096, 4096, 16), (16, 64, 4096, 16), (16, 4112, 4096, 32), (32, 8192, 2048, 32), (5, 12288, 768, 48)], ids=str)
def test_the_planner_takes_it(m, n, k, nr):
    assert check(None, m, n, k, True) == "skinny,sk=1" + (f",nr={nr}" if nr > 16 else "")


@pytest.mark.parametrize("nr", [16, 32, 48, 64])
@pytest.mark.parametrize("mr", [16, 32, 48, 64])
@pytest.mark.parametrize("m,n,k", [(17, 40, 8), (65, 136, 264), (96, 200, 1000), (130, 1032, 72), (70, 40, 2056)], ids=str)
def test_blocks_of_rows(m, n, k, mr, nr):
    """A last block of one row, of a part and of all of its rows; strips that are no whole number of XCDs."""
    for wv in ("", ",wv=8"):
        spec = f"skinny,sk=1{wv},nr={nr},mr={mr}"
        if wv and mr * nr > 2048:
            with pytest.raises(hg.HgemmError):
                hg.Plan(m, n, k, hg.Layouts.make(b_col_major=True), spec)
            continue
        assert check(spec, m, n, k, True) == spec
        check(spec, m, n, k, True, (8, 16, 8), (8, 8, 8), special=True)


@pytest.mark.parametrize("m,n,k,tile", [(17, 2048, 2056, (16, 16)), (33, 4096, 4096, (32, 32)), (96, 3000, 3072, (48, 32)), (320, 640, 3072, (32, 32))], ids=str)
def test_the_planner_takes_blocks_of_rows(m, n, k, tile):
    assert check(None, m, n, k, True) == "skinny,sk=1,nr=%d,mr=%d" % tile


@pytest.mark.parametrize("mr", [16, 32])
@pytest.mark.parametrize("m,n,k", [(16, 8, 8), (17, 40, 72), (65, 136, 264), (96, 200, 1000), (130, 1032, 520)], ids=str)
def test_row_major_b(m, n, k, mr):
    """Columns off the strip, K off a chunk and off the chunks of all waves, a last block of one row, of a part and of all of its rows."""
    spec = f"skinny,sk=1,nr=32,mr={mr}"
    assert check(spec, m, n, k, False) == spec
    check(spec, m, n, k, False, (8, 16, 8), (8, 8, 8), special=True)


@pytest.mark.parametrize("m,n,k,mr", [(17, 2048, 1408, 16), (64, 1920, 2048, 16), (96, 2504, 1776, 32), (128, 640, 2048, 16)], ids=str)
def test_the_planner_takes_it_for_row_major_b(m, n, k, mr):
    assert check(None, m, n, k, False) == f"skinny,sk=1,nr=32,mr={mr}"


@pytest.mark.parametrize("m,n,k", [(16, 4095, 4096), (1, 5118, 5120), (16, 11007, 4096)], ids=str)
def test_off_the_grid(m, n, k):
    """Next to streaming rows of the table: an odd C at any element's address, an A off the 16-byte grid (copied), B in strips where it lies, or copied
    because its base is not aligned."""
    for pads, offsets in (((8, 8, 5), (0, 8, 3)), ((1, 16, 0), (1, 0, 1)), ((0, 8, 1), (8, 3, 0))):
        got = check(None, m, n, k, True, pads, offsets)
        assert got.startswith("skinny,sk=1") and got.endswith("pad=1"), got
