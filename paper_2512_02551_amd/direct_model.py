"""Model behind hgemm_plan()'s choice between copying operands off the 16-byte grid and reading them where they lie.

    python -m paper_2512_02551_amd.direct_model gather --copies LIB --seed 21 --out FILE [--both]     # on the GPU
    python -m paper_2512_02551_amd.direct_model fit  [FILE ...]        # CPU; rewrites csrc/direct_model.inc
    python -m paper_2512_02551_amd.direct_model evaluate [FILE ...]    # CPU; the built library's choices

LIB is a build of the library from before it read such operands in place (commit 36f0870): its plans copy.  Timing files are JSON
lines of two kinds; csrc/direct_timings.jsonl.gz is the set the committed constants were fitted to.

    {"shape": [M, N, K], "tn": .., "copies": [spec, us], "direct": [[BM, BN, splits, fused, us], ...]}
        a random problem, every tile and split, operands in the last-level cache
    {"shape": [M, N, K], "tn": .., "ld": [lda, ldb, ldc], "copies": [spec, us from HBM, us from the cache], "direct": [the same]}
        (--both) the way that copies and the one that does not as it was planned then: random problems, and about twice as many
        where the choice was in doubt: a short K with a large C, one operand copied beside a long one that is not, a long unsplit K

direct_choice() in csrc/hgemm_api.hip holds the rule, predict_direct_us() there and predict_us() below are the same formula.
"""
from __future__ import annotations

import argparse
import gzip
import json
import os
import re

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
DATA = os.path.join(_HERE, "csrc", "direct_timings.jsonl.gz")
INC = os.path.join(_HERE, "csrc", "direct_model.inc")
CUS = 256
TILES = {(32, 64): "bm=32,bn=64,bk=64,wm=1,wn=2,st=4,pf=3", (64, 64): "bm=64,bn=64,bk=64,wm=2,wn=2,st=4,pf=3",
         (64, 128): "bm=64,bn=128,bk=64,wm=2,wn=2,st=4,pf=3", (128, 128): "bm=128,bn=128,bk=64,wm=2,wn=4,st=3,pf=3"}


def up8(v):
    return (v + 7) // 8 * 8


def features(shape, bm, bn, sk):
    """Workgroups per compute unit, K-tiles of a workgroup (whole pairs), splits that are not empty, MiB of planes."""
    M, N, K = shape
    kt = -(-K // 64)
    per = -(-kt // sk)
    eff = -(-kt // per)
    return -(-M // bm) * -(-N // bn) * eff / CUS, (per + 1) // 2 * 2, eff, M * N * 4 * eff / 2 ** 20


def predict_us(c, x, per, eff, mib, fused):
    """c: t0, wg, busy, flow, red2, red2_mib, red1, red1_mib of the tile."""
    w = np.ceil(x)
    t = c[0] + c[1] * w + per * ((c[2] * w) ** 4 + (c[3] * x) ** 4) ** 0.25
    return t + np.where(eff > 1, np.where(fused > 0, c[6] + c[7] * mib, c[4] + c[5] * mib), 0.0)


def load(paths):
    rows = []
    for p in paths:
        with (gzip.open if p.endswith(".gz") else open)(p, "rt") as f:
            rows += [json.loads(line) for line in f if line.strip()]
    return [r for r in rows if "ld" not in r], [r for r in rows if "ld" in r]


def spec_numbers(spec):
    d = {k: int(v) for k, v in re.findall(r"(\w+)=(\d+)", spec)}
    return d["bm"], d["bn"], d["sk"], d.get("fr", 0)


def copied_mb(shape, tn, lda=None, ldb=None):
    """MB read and written to copy the operands whose rows are not whole aligned chunks."""
    M, N, K = shape
    a = K % 8 or (lda or K) % 8
    b = (K if tn else N) % 8 or (ldb or 8) % 8
    return 4e-6 * ((M * up8(K) if a else 0) + (up8(N) * up8(K) if b else 0))


def fit(sweep, both):
    """Constants of every tile, of the copies, and what a K-tile takes longer from HBM.  Soft-L1 on log time."""
    import paper_2512_02551_amd as hg
    from scipy.optimize import least_squares

    tiles, errors = {}, {}
    for t in TILES:
        rows = []
        for r in sweep:
            best = min(d[4] for d in r["direct"])
            rows += [(*features(r["shape"], *t, d[2]), d[3], d[4]) for d in r["direct"] if tuple(d[:2]) == t and d[4] <= 1.8 * best]
        D = np.array(rows, dtype=float)

        def resid(p):
            return np.log(predict_us(np.abs(p), *D[:, :5].T)) - np.log(D[:, 5])

        starts = ([2.5, .4, .2, .2, 2, .3, 1., 1.5], [2, .4, .3, .3, 1, .3, 1, 1])
        q = min((least_squares(resid, s, loss="soft_l1", f_scale=0.1) for s in starts), key=lambda q: q.cost)
        tiles[t], errors[t] = np.abs(q.x), (len(rows), float(np.sqrt((resid(q.x) ** 2).mean())))
    rows = []
    for r in sweep:
        spec = r["copies"][0].replace(",pad=1", "")
        if spec.startswith("mfma") and copied_mb(r["shape"], r["tn"]):
            try:
                rows.append((hg.predict_us(r["shape"][0], up8(r["shape"][1]), up8(r["shape"][2]), spec), copied_mb(r["shape"], r["tn"]), r["copies"][1]))
            except hg.HgemmError:
                continue
    D = np.array(rows)
    q = least_squares(lambda p: np.log(p[0] + p[1] * D[:, 0] + p[2] * D[:, 1]) - np.log(D[:, 2]), [2, 1, .2], loss="soft_l1", f_scale=0.1)
    late = {}
    for t in TILES:                    # problems of 8 MB and more, one workgroup for a compute unit, eight K-tiles and more
        v = []
        for r in both:
            M, N, K = r["shape"]
            bm, bn, sk, _ = spec_numbers(r["direct"][0])
            x, per, _, _ = features(r["shape"], bm, bn, sk)
            if (bm, bn) == t and 2 * (M * r["ld"][0] + (N if r["tn"] else K) * r["ld"][1]) >= 8e6 and x <= 1 and per >= 8:
                v.append((r["direct"][1] - r["direct"][2]) / per)
        late[t] = float(np.quantile(v, 0.9))
    return tiles, q.x, late, errors


def write_inc(tiles, copies, late, note, path=INC):
    with open(path, "w") as f:
        f.write("// Constants of the model of kernels that read operands where they lie (predict_direct_us() in hgemm_api.hip).  Written by\n"
                f"// `python -m paper_2512_02551_amd.direct_model fit`; do not edit by hand.\n// {note}\n")
        for t, spec in TILES.items():
            f.write(f'DIRECT_TILE("mfma,{spec},sk=1,gm=8,di=1", {t[0]}, {t[1]}, ' + ", ".join(f"{v:.3f}" for v in [*tiles[t], late[t]]) + ")\n")
        f.write("DIRECT_COPIES(" + ", ".join(f"{v:.3f}" for v in copies) + ")\n")


def read_inc(path=INC):
    text = open(path).read()
    tiles = {(int(m[1]), int(m[2])): [float(v) for v in m[3].split(",")] for m in re.finditer(r'DIRECT_TILE\("[^"]*", (\d+), (\d+), ([^)]*)\)', text)}
    return tiles, [float(v) for v in re.search(r"DIRECT_COPIES\(([^)]*)\)", text)[1].split(",")]


def evaluate(both):
    import paper_2512_02551_amd as hg

    ratios = {True: [], False: []}
    for r in both:
        lay = hg.Layouts.make(r["tn"], *r["ld"])
        ratios[",di=1" in hg.plan_choice(*r["shape"], lay)].append([r["copies"][1] / r["direct"][1], r["copies"][2] / r["direct"][2]])
    for place, v in ratios.items():
        v = np.array(v)
        gm, slow = np.exp(np.log(v).mean(axis=0)), (v < 0.97).sum(axis=0)
        print(f"{len(v)} {'read in place' if place else 'copied'}: reading in place {gm[0]:.3f} times faster from HBM ({slow[0]} slower by more than 3 %, "
              f"the slowest {1 / v[:, 0].min():.2f} times), {gm[1]:.3f} from the cache ({slow[1]}, {1 / v[:, 1].min():.2f})")


def gather(seed, seconds, copies_lib, both, path):
    import ctypes
    import random
    import time

    import torch

    import paper_2512_02551_amd as hg

    hg.load()
    old = ctypes.CDLL(os.path.abspath(copies_lib))
    stream = torch.cuda.current_stream().cuda_stream
    rng = random.Random(seed)
    vp, i64 = ctypes.c_void_p, ctypes.c_int64

    def size(lo, hi, step=1):
        return int(min(max(round(lo * (hi / lo) ** rng.random() / step) * step, lo), hi))

    def problem():
        kind, tn = rng.random(), rng.randint(0, 1)
        if kind < 0.65:
            return size(65, 4200), size(65, 4200) | 1, size(129, 4200) | 1, tn
        if kind < 0.75:
            return size(33, 2000), size(65, 8000) | 1, size(64, 4200, 8), 0
        if kind < 0.85:
            return size(10, 2000), size(64, 8000, 8), size(64, 4200) | 1, tn
        return size(8, 64), size(65, 20000) | 1, size(64, 2000) | 1, tn

    t0 = time.time()
    with open(path, "w") as f:
        while time.time() - t0 < seconds:
            M, N, K, tn = problem()
            if M * N * K < 1 << 20:
                continue
            lay = hg.Layouts.make(b_col_major=bool(tn))
            n = max(3, min(64, int(6e8 // (2 * (M * K + N * K))))) if both else 3
            a = [torch.randint(-2, 3, (M, K), device="cuda").half() for _ in range(n)]
            b = [torch.randint(-2, 3, (N, K) if tn else (K, N), device="cuda").half() for _ in range(n)]
            c = torch.empty(M, N, device="cuda", dtype=torch.float16)
            arrays = [(vp * n)(*(t.data_ptr() for t in ts)) for ts in (a, b, [c] * n)]
            reps = max(6, min(100, int(1000 / (2 * M * N * K / 7e8 + 10))))

            def timed(run_many, sets):
                us = []
                for _ in range(6):
                    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
                    e0.record()
                    assert run_many(i64(reps), i64(sets)) == 0
                    e1.record()
                    e1.synchronize()
                    us.append(e0.elapsed_time(e1) / reps * 1e3)
                return round(float(np.median(us[1:])), 2)

            def times(lib, handle):
                def run_many(count, sets):
                    return lib.hgemm_run_many(handle, count, sets, i64(0), *arrays, vp(stream))
                return [timed(run_many, n), timed(run_many, 1)] if both else [timed(run_many, n)]

            handle, text = vp(), ctypes.create_string_buffer(512)
            assert old.hgemm_plan(ctypes.byref(handle), i64(M), i64(N), i64(K), ctypes.byref(lay)) == 0
            assert old.hgemm_plan_describe(handle, text, ctypes.c_size_t(512)) == 0
            row = {"shape": [M, N, K], "tn": bool(tn), "copies": [text.value.decode(), *times(old, handle)]}
            old.hgemm_destroy(handle)
            if both:
                with hg.Plan(M, N, K, lay) as p:
                    if "di=1" not in p.describe():
                        continue
                    row.update(ld=[K, K if tn else N, N], direct=[p.describe().replace(",pad=1", ""), *times(hg.load(), p._h)])
            else:
                row["direct"] = []
                for (bm, bn), spec in TILES.items():
                    tiles, kt = -(-M // bm) * -(-N // bn), -(-K // 64)
                    for sk in (1, 2, 3, 4, 6, 8, 12, 16):
                        if sk > 1 and (tiles * sk > 1024 or kt // sk < 2 or tiles > CUS):
                            break
                        for fr in (0, 1):
                            if fr and (sk == 1 or sk * M * N * 4 > 6 << 20):
                                continue
                            with hg.Plan(M, N, K, lay, f"mfma,{spec},sk={sk},gm=8{',fr=1' if fr else ''},di=1") as p:
                                row["direct"].append([bm, bn, sk, fr, *times(hg.load(), p._h)])
            f.write(json.dumps(row) + "\n")
            f.flush()


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    sub = ap.add_subparsers(dest="cmd", required=True)
    g_ = sub.add_parser("gather")
    g_.add_argument("--copies", required=True, metavar="LIB")
    g_.add_argument("--seed", type=int, required=True)
    g_.add_argument("--seconds", type=float, default=300)
    g_.add_argument("--both", action="store_true")
    g_.add_argument("--out", required=True)
    for name in ("fit", "evaluate"):
        sub.add_parser(name).add_argument("files", nargs="*", default=[DATA])
    args = ap.parse_args()
    if args.cmd == "gather":
        gather(args.seed, args.seconds, args.copies, args.both, args.out)
    elif args.cmd == "fit":
        sweep, both = load(args.files)
        tiles, copies, late, errors = fit(sweep, both)
        write_inc(tiles, copies, late, f"{sum(n for n, _ in errors.values())} timings of {len(sweep)} problems, rms "
                  + ", ".join(f"{100 * e:.1f}" for _, e in errors.values()) + f" %; from HBM: {len(both)} problems.")
        print(open(INC).read())
    else:
        evaluate(load(args.files)[1])
