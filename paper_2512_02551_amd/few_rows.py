"""Measured problems behind hgemm_plan()'s choice for up to 32 rows of A that are not in the dispatch table.

Decoding multiplies a handful of rows by weights that come from HBM.  The cost model of plan_model.py is fitted to operands in
the last-level cache and to one schedule of each family; here random problems of that kind are timed with every kernel that may be
the fastest, and csrc/few_rows.inc holds for each the kernels that are close to the fastest.  few_rows_choice() in csrc/hgemm_api.hip
looks up the nearest.

    python -m paper_2512_02551_amd.few_rows gather --seed 1 --seconds 500 --out FILE [--against LIB]   # on the GPU
    python -m paper_2512_02551_amd.few_rows recheck --out FILE [--against LIB] [FILE]       # on the GPU; every problem of a check file again
    python -m paper_2512_02551_amd.few_rows build [FILE ...]          # CPU; rewrites csrc/few_rows.inc
    python -m paper_2512_02551_amd.few_rows evaluate [--against LIB] [FILE ...]     # CPU; the built library's choices

csrc/few_rows_timings.jsonl.gz, which the committed rows are built from, holds 8390 problems of up to 32 rows (row-major B: 40; those of
more than 32 count as neighbours in a mean, but make no rows): three quarters products of transformer layers (widths 1024-8192 in
steps of 128, feed-forward widths 2.5-4 times that), the others output heads (8000-64000 columns, K 512-8192).  All candidates,
operands from HBM (rotated through 800 MB); its first line names the kernels, the others are {"shape": [M, N, K], "tn": B column-major,
"us": [[kernel, us], ...]}.  Resident A was timed afterwards, beside the kernel that was chosen then, and stands with its time over that
one's, on K from 1200 on only: on a shorter K it wins less than 5 % from HBM and loses as much from the cache (1 x 18352 x 808:
10.3 -> 8.2 us, 4.9 -> 6.3).

csrc/few_rows_check.jsonl.gz holds 4885 other problems as `gather` writes them, which the choices are checked on: half products of
layers, a quarter output heads, a quarter any multiples of 8; {"shape", "tn", "cands": [[kernel, us from HBM, us from the cache], ...]} with
the kernels whose first timing was within a fifth of the fastest, the library's choice and that of the builds it is compared with
(--against: another build of the library, of an earlier commit, say).  The 1373 that run on strips of B through LDS were timed again since;
the others stand as first timed, 438 of them with streaming kernels of a column-major B as they were before, when lanes loaded operands (a spec without nr then meant strips
of 16 rows of B, now of up to 48).  With every problem timed again (`recheck`) the choices are 6 and 8 % from the fastest kernel, not 5 and 7.
csrc/few_rows_timings.jsonl.gz has that family's kernels as they were before.
"""
from __future__ import annotations

import argparse
import ctypes
import gzip
import json
import math
import os
import re

import numpy as np

_HERE = os.path.dirname(os.path.abspath(__file__))
DATA = os.path.join(_HERE, "csrc", "few_rows_timings.jsonl.gz")
CHECK = os.path.join(_HERE, "csrc", "few_rows_check.jsonl.gz")
INC = os.path.join(_HERE, "csrc", "few_rows.inc")

# Tiles of 32 rows; the streaming family's kernels come from hgemm_candidates().
TILES = ["bm=32,bn=64,bk=64,wm=1,wn=2,st=4,pf=3", "bm=32,bn=128,bk=64,wm=1,wn=4,st=4,pf=3", "bm=32,bn=128,bk=128,wm=1,wn=4,st=4,pf=3",
         "bm=32,bn=192,bk=64,wm=1,wn=2,st=4,pf=3", "bm=32,bn=256,bk=64,wm=1,wn=4,st=4,pf=3"]


def number(spec: str, key: str, default: int = 0) -> int:
    m = re.search(rf"\b{key}=(\d+)", spec)
    return int(m[1]) if m else default


def problem(rng):
    """Half the products of a transformer layer and a quarter output heads, at widths in use, and a quarter any multiples of 8."""
    def size(lo, hi, step=1):
        return int(min(max(round(lo * (hi / lo) ** rng.random() / step) * step, lo), hi))

    M, tn, kind = size(1, 32), rng.random() < 0.5, rng.random()
    if kind < 0.5:
        w = size(1024, 8192, 128)
        up = int(w * rng.uniform(2.5, 4.0)) // 128 * 128
        N, K = rng.choice([(w, w), (up, w), (w, up), (up + w, w)])
    elif kind < 0.75:
        N, K = size(8000, 160000, 8), size(512, 8192, 8)
    else:
        N, K = size(512, 65536, 8), size(512, 16384, 8)
    return (M, N, K, tn) if N * K <= 1 << 29 else problem(rng)


def choice(path, M, N, K, tn):
    """What a build of the library runs the problem on (None: the package's own build)."""
    import paper_2512_02551_amd as hg

    lay = hg.Layouts.make(b_col_major=tn)
    if path is None:
        return hg.plan_choice(M, N, K, lay).split(": ", 1)[1]
    hg.load()          # binds the HIP runtime that both builds then share
    i64, buf = ctypes.c_int64, ctypes.create_string_buffer(512)
    assert ctypes.CDLL(os.path.abspath(path)).hgemm_plan_choice(i64(M), i64(N), i64(K), ctypes.byref(lay), buf, ctypes.c_size_t(512)) == 0
    return buf.value.decode().split(": ", 1)[1]


def specs_to_time(hg, M, N, K, tn):
    out = []
    for t in TILES:
        tiles, ksteps = -(-N // number(t, "bn")), -(-K // number(t, "bk"))
        for sk in (1, 2, 3, 4, 6, 8, 12, 16):
            if sk > 1 and (ksteps // sk < 2 or tiles * sk > 2048 or sk * M * N * 4 > 24 << 20):
                break
            out.append(f"mfma,{t},sk={sk},gm=8")
            if sk > 1 and sk * M * N * 4 <= 3 << 20:
                out.append(out[-1] + ",fr=1")
    out += [s for s in hg.candidates(M, N, K, hg.Layouts.make(b_col_major=tn)) if s.startswith("skinny") and "wv=16" not in s and (not tn or number(s, "sk") == 1)]
    return out


def gather(seed: int, seconds: float, path: str, against):
    import random
    import time

    import torch

    import paper_2512_02551_amd as hg

    hg.load()
    sh = torch.cuda.current_stream().cuda_stream
    rng = random.Random(seed)
    pool = torch.empty(3 << 28, dtype=torch.float16, device="cuda")           # operand sets are cut from here
    part = torch.randn(1 << 26, device="cuda").mul_(0.02).half()
    for i in range(0, pool.numel(), part.numel()):
        pool[i:i + part.numel()] = part
    c = torch.empty(32 * 160000, dtype=torch.float16, device="cuda")

    def timed(p, sets, reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        p.run_many(reps, sets, sh)          # all sets have one C: every call is a launch of its own
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / reps * 1e3

    t0, done = time.time(), 0
    with open(path, "w") as f:
        while time.time() - t0 < seconds:
            M, N, K, tn = problem(rng)
            lay = hg.Layouts.make(b_col_major=tn)
            elems = (M * K + 127) // 128 * 128 + N * K
            n = max(1, min(64, pool.numel() // elems, int(6e8 // (2 * elems)) + 1))
            assert n * elems <= pool.numel() and M * N <= c.numel(), (M, N, K)
            base = pool.data_ptr()
            sets = [(base + 2 * i * elems, base + 2 * (i * elems + elems - N * K), c.data_ptr()) for i in range(n)]
            first, plans = {}, {}
            chosen = [choice(lib, M, N, K, tn) for lib in [None] + against]
            for s in dict.fromkeys(chosen + specs_to_time(hg, M, N, K, tn)):
                try:
                    p = hg.Plan(M, N, K, lay, s)
                except hg.HgemmError:
                    continue
                if p.describe() == s:
                    timed(p, sets, 2)
                    first[s] = timed(p, sets, 12)
                    if s in chosen or first[s] <= 1.2 * min(first.values()):
                        plans[s] = p
                        continue
                p.destroy()
            near = [s for s in plans if s in chosen or first[s] <= 1.2 * min(first.values())]
            times = {s: ([], []) for s in near}
            reps = max(4, min(60, int(300 / min(first.values()))))
            for _ in range(5):
                for s in near:
                    times[s][0].append(timed(plans[s], sets, reps))
            for _ in range(5):
                for s in near:
                    times[s][1].append(timed(plans[s], sets[:1], reps))
            for p in plans.values():
                p.destroy()
            cands = [[s] + [round(float(np.median(v[1:])), 2) for v in times[s]] for s in near]
            f.write(json.dumps({"seed": seed, "shape": [M, N, K], "tn": tn, "cands": cands}) + "\n")
            f.flush()
            done += 1
            if done % 50 == 0:
                print(f"{done} problems, {time.time() - t0:.0f} s", flush=True)


def recheck(src: str, path: str, against):
    """Every problem of `src` again: the kernels that stand there and the library's choice."""
    import torch

    import paper_2512_02551_amd as hg

    rows = load([src])
    pool = torch.randn(1 << 26, device="cuda").mul_(0.02).half().repeat(12)
    c = torch.empty(32 * 160000, dtype=torch.float16, device="cuda")
    sh = torch.cuda.current_stream().cuda_stream

    def timed(p, sets, reps):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        p.run_many(reps, sets, sh)
        e1.record()
        e1.synchronize()
        return e0.elapsed_time(e1) / reps * 1e3

    done = 0
    for r in rows:
        M, N, K = r["shape"]
        specs = list(dict.fromkeys([choice(lib, M, N, K, r["tn"]) for lib in [None] + against] + [x[0] for x in r["cands"]]))
        elems = (M * K + 127) // 128 * 128 + N * K
        n = max(1, min(64, pool.numel() // elems, int(6e8 // (2 * elems)) + 1))
        assert n * elems <= pool.numel() and M * N <= c.numel(), (M, N, K)
        sets = [(pool.data_ptr() + 2 * i * elems, pool.data_ptr() + 2 * (i * elems + elems - N * K), c.data_ptr()) for i in range(n)]
        plans = [hg.Plan(M, N, K, hg.Layouts.make(b_col_major=r["tn"]), s) for s in specs]
        reps = max(4, min(60, int(300 / timed(plans[0], sets, 4))))
        times = [[[], []] for _ in plans]
        for w, some in ((0, sets), (1, sets[:1])):
            for _ in range(5):
                for p, t in zip(plans, times):
                    t[w].append(timed(p, some, reps))
        r["cands"] = [[s] + [round(float(np.median(v[1:])), 2) for v in t] for s, t in zip(specs, times)]
        for p in plans:
            p.destroy()
        done += 1
        if done % 100 == 0:
            print(f"{done} problems", flush=True)
    with gzip.open(path, "wt", compresslevel=9) as f:
        f.writelines(json.dumps(r) + "\n" for r in rows)


def load(paths):
    rows = []
    for p in paths:
        specs = None
        with (gzip.open if p.endswith(".gz") else open)(p, "rt") as f:
            for line in f:
                r = json.loads(line)
                if "specs" in r:
                    specs = r["specs"]
                    continue
                if specs:
                    r["cands"] = [[specs[i], us, None] for i, us in r.pop("us")]
                else:       # slower from the cache than from HBM: the host was late with a launch
                    r["cands"] = [[c, hbm, min(hbm, cache)] for c, hbm, cache in r["cands"]]
                rows.append(r)
    return rows


NEIGHBOURS, WITHIN, LISTED, REACH = 10, 1.03, 5, 0.3


def columns(n):
    return np.minimum(3, -(-n // 16384))


def build(rows):
    """Per layout: [(shape, [specs, best first])].  The list of a problem comes from its ten nearest neighbours, itself among them: the
    kernels' times over the fastest (2 at most), nearer ones weighted more.  Problems that a kept neighbour speaks for are left
    out, and in the end those that no lookup may reach: of more than 32 rows, and of a row-major B of 256 MiB and more, which is streamed."""
    import random

    out = {}
    for tn in (False, True):
        sel = [r for r in rows if r["tn"] == tn]
        logs = np.array([[math.log2(v) for v in r["shape"]] for r in sel])
        part = np.array([columns(r["shape"][1]) for r in sel])
        weights = np.array([0.3, 1.0, 1.0])
        relative = []
        for r in sel:
            best = min(c[1] for c in r["cands"])
            relative.append({c[0]: min(c[1] / best, 2.0) for c in r["cands"] if "bm=64" not in c[0]})

        def distances(i, to):
            """few_rows_choice()'s measure."""
            return np.abs(logs[to] - logs[i]) @ weights + 0.25 * (part[to] != part[i])

        every, lists = np.arange(len(sel)), []
        for i in range(len(sel)):
            d = distances(i, every)
            near = np.argsort(d, kind="stable")[:NEIGHBOURS]
            score, weight, total = {}, {}, 0.0
            for j in near:
                w = 1.0 / (0.05 + d[j])
                total += w
                for s, v in relative[j].items():
                    score[s] = score.get(s, 0.0) + w * v
                    weight[s] = weight.get(s, 0.0) + w
            ranked = sorted((score[s] / weight[s], s) for s in score if weight[s] > 0.6 * total)
            lists.append([s for v, s in ranked if v <= ranked[0][0] * WITHIN][:LISTED])
        order = list(range(len(sel)))
        random.Random(3).shuffle(order)
        kept = []
        for i in order:
            if kept:
                d = distances(i, np.array(kept))
                j = kept[int(np.argmin(d))]
                if d.min() < 0.2 and lists[j][0] == lists[i][0] and 2 * len(set(lists[i]) & set(lists[j])) >= min(len(lists[i]), len(lists[j])):
                    continue
            kept.append(i)
        reached = [i for i in kept if sel[i]["shape"][0] <= 32 and (tn or 2.0 * sel[i]["shape"][1] * sel[i]["shape"][2] < 2 ** (28 + REACH))]
        out[tn] = sorted((tuple(sel[i]["shape"]), lists[i]) for i in reached)
    return out


def columns_quarter(n):
    """The order the rows are searched in: quarters of an octave of N, K in each."""
    top = n.bit_length() - 1
    return 4 * top + ((n << 2 >> top) & 3)


def write(table, note, path=INC):
    specs = sorted({s for rows in table.values() for _, l in rows for s in l})
    text = ["// Problems of up to 32 rows of A that were timed: rows, columns, K, and the specialisations within 3 % of the best, best first (numbers of",
            "// kFewSpecs, -1: none).  Written by `python -m paper_2512_02551_amd.few_rows build`; do not edit by hand.", f"// {note}",
            "static const char* const kFewSpecs[] = {", *(f'    "{s}",' for s in specs), "};"]
    for tn, name in ((False, "kFewRowsNN"), (True, "kFewRowsTN")):
        text.append(f"static const FewRow {name}[] = {{")
        line = "   "
        for (m, n, k), l in sorted(table[tn], key=lambda r: (columns_quarter(r[0][1]), r[0][2], r[0])):
            item = f" {{{m}, {n}, {k}, {{{', '.join(str(specs.index(s)) for s in l)}{', -1' * (LISTED - len(l))}}}}},"
            if len(line) + len(item) > 150:
                text.append(line)
                line = "   "
            line += item
        text += [line, "};"]
    with open(path, "w") as f:
        f.write("\n".join(text) + "\n")


def mean(v):
    return math.exp(float(np.mean(np.log(v)))) if len(v) else float("nan")


def report(rows, chosen, before):
    """`chosen` and `before`: per problem a spec, or None.  Times of the one over the other, and over the fastest."""
    for w, name in ((1, "from HBM"), (2, "from the cache")):
        best, gain = [], []
        for r, s, b in zip(rows, chosen, before):
            t = {c[0]: c[w] for c in r["cands"]}
            if s not in t or b not in t:
                continue
            best.append(t[s] / min(t.values()))
            if s != b:
                gain.append(t[b] / t[s])
        slow = [sum(g < x for g in gain) for x in (0.97, 0.9)]
        print(f"{name}: {len(best)} problems, {mean(best):.4f} of the fastest; {len(gain)} choices differ, {mean(gain):.4f} times faster, {slow[0]} slower by more than 3 %, {slow[1]} by 10 %")


if __name__ == "__main__":
    ap = argparse.ArgumentParser()
    sub = ap.add_subparsers(dest="cmd", required=True)
    g_ = sub.add_parser("gather")
    g_.add_argument("--seed", type=int, required=True)
    g_.add_argument("--seconds", type=float, default=500)
    g_.add_argument("--out", required=True)
    g_.add_argument("--against", action="append", default=[], metavar="LIB")
    b_ = sub.add_parser("build")
    b_.add_argument("files", nargs="*", default=[DATA])
    e_ = sub.add_parser("evaluate")
    e_.add_argument("--against", default=None, metavar="LIB")
    e_.add_argument("files", nargs="*", default=[CHECK])
    r_ = sub.add_parser("recheck")
    r_.add_argument("--out", required=True)
    r_.add_argument("--against", action="append", default=[], metavar="LIB")
    r_.add_argument("file", nargs="?", default=CHECK)
    args = ap.parse_args()
    if args.cmd == "recheck":
        recheck(args.file, args.out, args.against)
    elif args.cmd == "build":
        rows = load(args.files)
        table = build(rows)
        write(table, f"From {len(rows)} random problems, each row the mean of the {NEIGHBOURS} nearest; problems that a kept neighbour speaks for are left out.")
        print(len(rows), "problems,", {("tn" if t else "nn"): len(v) for t, v in table.items()}, "rows")
    elif args.cmd == "evaluate":
        rows = load(args.files)
        chosen = [choice(None, *r["shape"], r["tn"]) for r in rows]
        report(rows, chosen, [choice(args.against, *r["shape"], r["tn"]) for r in rows] if args.against else chosen)
    elif args.cmd == "gather":
        gather(args.seed, args.seconds, args.out, args.against)
