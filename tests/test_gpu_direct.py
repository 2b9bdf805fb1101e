"""The kernels that read operands off the 16-byte grid where they lie, through registers (spec key di=1)."""
import itertools

import pytest
import torch

import paper_2512_02551_amd as hg

pytestmark = pytest.mark.gpu

TILES = {(32, 64): "bm=32,bn=64,bk=64,wm=1,wn=2,st=4,pf=3", (64, 64): "bm=64,bn=64,bk=64,wm=2,wn=2,st=4,pf=3",
         (64, 128): "bm=64,bn=128,bk=64,wm=2,wn=2,st=4,pf=3", (128, 128): "bm=128,bn=128,bk=64,wm=2,wn=4,st=3,pf=3"}


def embedded(rows, cols, ld, offset, g, fill="int"):
    """A rows x cols matrix of small integers with pitch ld, `offset` elements into a buffer that is NaN everywhere else: in
    front of it, between its rows and right behind its last element, where the buffer ends."""
    buf = torch.full((offset + (rows - 1) * ld + cols,), float("nan"), dtype=torch.float16, device="cuda")
    view = torch.as_strided(buf, (rows, cols), (ld, 1), offset)
    view.copy_(torch.randint(-2, 3, (rows, cols), generator=g, device="cuda"))
    return buf, view


def check(spec, M, N, K, tn, pads=(0, 0, 0), offsets=(0, 0, 0), special=False):
    g = torch.Generator(device="cuda").manual_seed(M * 31 + N * 7 + K)
    lda, ldb, ldc = K + pads[0], (K if tn else N) + pads[1], N + pads[2]
    abuf, a = embedded(M, K, lda, offsets[0], g)
    bbuf, b = embedded(*((N, K) if tn else (K, N)), ldb, offsets[1], g)
    if special:
        a[M // 2, K - 1] = float("inf")
        a[0, 0] = float("nan")
        (b[N - 1] if tn else b[:, N - 1])[K // 2] = float("-inf")
    cbuf = torch.full((offsets[2] + M * ldc + 16,), float("nan"), dtype=torch.float16, device="cuda")
    c = torch.as_strided(cbuf, (M, N), (ldc, 1), offsets[2])
    af, bf = a.cpu().double(), b.cpu().double()
    ref = (af @ (bf.t().contiguous() if tn else bf)).half()             # sums of less than 2^24: exact in fp32, rounded once
    with hg.Plan(M, N, K, hg.Layouts.make(b_col_major=tn, lda=lda, ldb=ldb, ldc=ldc), spec) as p:
        what = f"{M}x{N}x{K} {'tn' if tn else 'nn'} pads={pads} offsets={offsets} {p.describe()}"
        for _ in range(2):                                              # the second time on counters the first one left
            cbuf.fill_(float("nan"))
            p.run(abuf.data_ptr() + 2 * offsets[0], bbuf.data_ptr() + 2 * offsets[1], cbuf.data_ptr() + 2 * offsets[2], torch.cuda.current_stream().cuda_stream)
            torch.cuda.synchronize()
            got = c.cpu()
            assert torch.equal(torch.isnan(got), torch.isnan(ref)), what
            assert torch.equal(torch.nan_to_num(got, nan=0.0), torch.nan_to_num(ref, nan=0.0)), what
            assert int(torch.isnan(cbuf).sum()) == cbuf.numel() - M * N + int(torch.isnan(ref).sum()), what + ": wrote outside C"
        return p.describe()


@pytest.mark.parametrize("tn", [False, True], ids=["nn", "tn"])
@pytest.mark.parametrize("tile", TILES, ids=str)
def test_direct_kernels_at_the_edges_of_their_tiles(tile, tn):
    """One element less and more than whole tiles and K-tiles, the smallest operands, odd and even numbers of K-tiles; C, A and B at any
    element's address and pitch; NaN around and between the rows of all three."""
    bm, bn = tile
    spec = f"mfma,{TILES[tile]},sk=1,gm=8,di=1"
    sizes = [(1, 8, 8), (bm, bn, 64), (bm + 1, bn + 1, 65), (bm - 1, bn - 1, 63), (2 * bm + 1, 2 * bn - 1, 129), (bm, 2 * bn + 9, 191), (3, bn + 7, 193), (bm + 5, 9, 257)]
    for (M, N, K), (pads, offsets) in itertools.product(sizes, [((0, 0, 0), (0, 0, 0)), ((1, 3, 5), (1, 3, 5)), ((8, 16, 8), (7, 8, 2))]):
        check(spec, M, N, K, tn, pads, offsets)
    check(spec, bm + 3, bn + 5, 201, tn, (3, 1, 2), (1, 1, 1), special=True)


@pytest.mark.parametrize("tn", [False, True], ids=["nn", "tn"])
@pytest.mark.parametrize("tile", TILES, ids=str)
def test_direct_kernels_split_over_k(tile, tn):
    """Two-launch and fused splits: last ranges of one element, of one K-tile and of an odd number of K-tiles."""
    bm, bn = tile
    for (M, N, K), sk, fr in itertools.product([(bm + 1, bn + 3, 129), (7, 2 * bn + 1, 64 * 5 + 1), (bm, bn, 64 * 7 - 1), (bm + 2, 11, 1003)], (2, 3, 4), ("", ",fr=1")):
        check(f"mfma,{TILES[tile]},sk={sk},gm=8{fr},di=1", M, N, K, tn, (1, 1, 1), (1, 3, 1), special=K == 1003)


@pytest.mark.parametrize("M,N,K,tn", [(65, 65, 257, False), (500, 501, 503, True), (1000, 1001, 1003, False), (2000, 2001, 1001, False), (90, 71, 4101, True), (40, 4215, 1245, True),
                                      (300, 303, 304, False), (201, 1000, 999, True)])
def test_planned_problems_off_the_16_byte_grid_that_are_read_where_they_lie(M, N, K, tn):
    """What the planner takes these kernels for, with bases at any element's address."""
    for pads, offsets in (((0, 0, 0), (0, 0, 0)), ((3, 5, 1), (1, 2, 3))):
        desc = check(None, M, N, K, tn, pads, offsets)
        assert ",di=1" in desc and desc.endswith(",pad=1"), desc


def test_direct_kernels_refuse_what_their_loads_cannot_read():
    for M, N, K in ((64, 7, 64), (64, 64, 7)):
        with pytest.raises(hg.HgemmError) as e:
            hg.Plan(M, N, K, None, f"mfma,{TILES[(64, 64)]},sk=1,gm=8,di=1")
        assert e.value.status == 2
