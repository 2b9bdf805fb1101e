"""Fused split-K: the workgroup that arrives last sums the planes of all.  A plane that has not arrived would leave the one of the launch before,
so launches alternate between operands whose results differ everywhere."""
import pytest
import torch

import paper_2512_02551_amd as hg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m,n,k,tn,spec", [
    (7, 10352, 4120, False, "mfma,bm=32,bn=128,bk=64,wm=1,wn=4,st=4,pf=3,sk=2,gm=8,fr=1"), (1, 4096, 4096, False, "mfma,bm=32,bn=64,bk=64,wm=1,wn=2,st=4,pf=3,sk=8,gm=8,fr=1"),
    (32, 2048, 8192, True, "mfma,bm=32,bn=128,bk=128,wm=1,wn=4,st=4,pf=3,sk=6,gm=8,fr=1"), (256, 256, 4096, False, "mfma,bm=64,bn=64,bk=64,wm=2,wn=2,st=4,pf=3,sk=16,gm=8,fr=1"),
    (200, 264, 2000, True, "mfma,bm=128,bn=128,bk=64,wm=2,wn=4,st=3,pf=3,sk=4,gm=8,fr=1"), (131, 257, 1999, False, "mfma,bm=64,bn=64,bk=64,wm=2,wn=2,st=4,pf=3,sk=5,gm=8,fr=1,di=1"),
    (16, 4096, 8192, False, "skinny,sk=8,fr=1"), (40, 1032, 4096, False, "skinny,sk=4,fr=1,wv=8"), (16, 4096, 8192, True, "skinny,sk=4,fr=1,wv=8"), (33, 1000, 4096, True, "skinny,sk=3,fr=1,nr=32")],
    ids=lambda v: v if isinstance(v, str) else str(v))
def test_no_plane_of_the_launch_before_is_summed(m, n, k, tn, spec):
    g = torch.Generator(device="cuda").manual_seed(m + n + k)
    sh = torch.cuda.current_stream().cuda_stream
    b = torch.randint(-1, 2, (n, k) if tn else (k, n), generator=g, device="cuda").half()
    sets = []
    for _ in range(2):
        a = torch.randint(-1, 2, (m, k), generator=g, device="cuda").half()
        bf = b.cpu().float()                                           # sums of at most 8192 in magnitude: exact in float32
        sets.append((a, (a.cpu().float() @ (bf.t().contiguous() if tn else bf)).half().cuda()))
    c = torch.empty((m, n), dtype=torch.float16, device="cuda")
    wrong = torch.zeros((), dtype=torch.int64, device="cuda")
    with hg.Plan(m, n, k, hg.Layouts.make(b_col_major=tn), spec) as p:
        assert ",fr=1" in p.describe()
        for i in range(200):
            a, ref = sets[i % 2]
            p.run(a.data_ptr(), b.data_ptr(), c.data_ptr(), sh)
            wrong += (c != ref).sum()
        assert int(wrong) == 0, p.describe()
