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
