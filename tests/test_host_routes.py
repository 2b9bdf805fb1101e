"""Which way a call goes -- what it allocates and launches, what it refuses -- read from the host code on a machine
without a GPU (fake_hip.py)."""
import os
import re

import pytest

import paper_2512_02551_amd as hg
from fake_hip import ask

CSRC = os.path.join(os.path.dirname(os.path.abspath(hg.__file__)), "csrc")


def table_rows(tn):
    text = open(os.path.join(CSRC, "dispatch_table_tn.inc" if tn else "dispatch_table.inc")).read()
    rows = [(tuple(int(v) for v in m[:3]), m[3]) for m in re.findall(r'\{\s*(\d+),\s*(\d+),\s*(\d+),\s*"([^"]*)"', text)]
    rows = [r for r in rows if min(r[0]) > 0 and r[1]]
    assert len(rows) > 1000
    return rows


@pytest.mark.parametrize("tn", [False, True])
def test_the_static_entry_point_runs_every_table_row_whose_workspace_fits(tn):
    """A workspace of up to HGEMM_STATIC_SCRATCH_BYTES, that size included: the launches of the planned call."""
    shapes = [s for s, _ in table_rows(tn)]
    full = 0
    for (m, n, k), r in zip(shapes, ask([{"M": m, "N": n, "K": k, "tn": tn} for m, n, k in shapes])):
        assert r["plan"] == 0 and r["run"] == 0
        if r["workspace"] > hg.STATIC_SCRATCH_BYTES:
            continue
        full += r["workspace"] == hg.STATIC_SCRATCH_BYTES
        assert r["static"] == 0, (m, n, k, r["describe"], r["workspace"])
        assert r["static_log"] == r["run_log"], (m, n, k, r["describe"])
    assert full > 0


def kernels(log):
    """Names and grids of the launches of a log."""
    out = []
    for line in log:
        if line.startswith("launch "):
            _, name, x, y = line.split()
            out.append((re.search(r"([a-z0-9_]+_kernel)", re.sub(r"^_ZN5hgemm\d+", "", name))[1], int(x), int(y)))
    return out


@pytest.mark.parametrize("tn", [False, True])
@pytest.mark.parametrize("m,n,k", [(3, 1001, 1003), (2, 4099, 520), (266, 360, 280), (100, 1001, 1008)])
def test_a_pitch_of_c_beyond_32_bits_keeps_the_matrix_core_kernels(m, n, k, tn):
    """Rows of C 2^31 elements apart and more: stored packed and copied from there; one row: stored in place."""
    qs = [{"M": rows, "N": n, "K": k, "tn": tn, "ldc": (1 << 31) + pad} for rows in (m, 1) for pad in (3, 1 << 31)]
    qs.append({"M": m, "N": n, "K": k, "tn": tn, "ldc": (1 << 31) - 1})
    for q, r in zip(qs, ask(qs)):
        if q["M"] * n * k < 1 << 20:
            assert r["describe"] == "generic"
            continue
        names = [name for name, _, _ in kernels(r["run_log"])]
        assert r["run"] == 0 and "generic_gemm_kernel" not in names, (q, names)
        assert ("copy_back_kernel" in names) == (q["M"] > 1 and q["ldc"] >= 1 << 31), (q, names)
        assert r["static"] == 0 and r["static_log"] == r["run_log"], q
